// contraction.hip -- the information matrix as two symmetric rank-K products,
// and the FP64 Cholesky solve of a Newton step (gfx950).
//
//   I = X' diag(b) X - Z'Z,   b_r = w_r Lambda_r,   Z_gj = sqrt(d_g) xbar_gj
// (the Hessian of Eq. strat_h with the order of its sums exchanged; see
// newton.hip).  Both products have the form C = sum_k c_k u_k u_k' over K
// rows with u_k in R^p stored column-wise ([p][ld], k contiguous).
//
// FP64 reference kernel: 64x64 tiles of the upper triangle, K split across
// workgroups, 32-row chunks staged in LDS, each thread owning a 4x4 block;
// the split partials are summed in split order (deterministic).
//
// BF16 kernel (matrix cores): u is stored as BF16 with a power-of-two scale
// per column; v_mfma_f32_32x32x16_bf16 accumulates 32x32 tiles in FP32.  The
// weights c_k multiply one operand in FP32 before it is rounded to BF16.
// A workgroup's waves share one K range and the tiles of the upper triangle (p <= 256) or of one
// 256 x 256 block of it, and the FP32 partials of the K ranges are summed in FP64
// in range order with the column scales applied.
#include <hip/hip_bf16.h>
#include <math.h>

#include "internal.h"
#include "newton.h"

namespace coxmi {

namespace {

constexpr int kTile = 64, kKc = 32, kSyrkThreads = 256, kWaveC = 64;

// x of lane src, for a src that is the same in every lane of the wave (two v_readlane, no
// trip through the LDS crossbar as for a per-lane source)
__device__ __forceinline__ double lane_value(double x, int src)
{
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), src);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

__device__ __forceinline__ void tile_pair(int pair, int nt, int &ti, int &tj)
{
    // pairs (ti <= tj) in row-major order of the upper triangle
    int i = 0, rem = pair;
    while (rem >= nt - i) {
        rem -= nt - i;
        ++i;
    }
    ti = i;
    tj = i + rem;
}

// (K range, group) of a workgroup of a (splits, groups) grid.  Workgroups go to the 8 XCDs in
// turn by linear id; when splits is a multiple of 8 the ids are renumbered so that every group
// of one K range runs on one XCD at nearly the same time, and the rows of the range that each
// of them stages are read from HBM once and from that XCD's L2 after.  Only the assignment of
// work to workgroups changes, not the work.
__device__ __forceinline__ void split_group(int &split, int &group)
{
    const int nsplit = gridDim.x, ngroup = gridDim.y;
    if (ngroup == 1 || nsplit % 8 != 0) {
        split = blockIdx.x;
        group = blockIdx.y;
        return;
    }
    const int L = blockIdx.x + nsplit * blockIdx.y;
    const int x = L % 8, r = L / 8;
    split = x + 8 * (r / ngroup);
    group = r % ngroup;
}


__global__ __launch_bounds__(kSyrkThreads) void syrk_f64_kernel(const double *u, int64_t ldu, int p,
                                                                const double *c, int64_t K, int64_t kchunk,
                                                                double *part)
{
    __shared__ double As[kTile][kKc + 1];
    __shared__ double Bs[kTile][kKc + 1];
    const int nt = (p + kTile - 1) / kTile;
    const int npairs = nt * (nt + 1) / 2;
    const int pair = blockIdx.x, s = blockIdx.y;
    int ti, tj;
    tile_pair(pair, nt, ti, tj);
    const int t = threadIdx.x, tx = t % 16, ty = t / 16;
    const int64_t k0 = (int64_t)s * kchunk;
    const int64_t k1 = k0 + kchunk < K ? k0 + kchunk : K;
    double acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int bb = 0; bb < 4; ++bb) acc[a][bb] = 0.0;
    for (int64_t k = k0; k < k1; k += kKc) {
#pragma unroll
        for (int e = 0; e < kTile * kKc / kSyrkThreads; ++e) {
            const int idx = t + kSyrkThreads * e;
            const int i = idx / kKc, kk = idx % kKc;
            const int64_t kr = k + kk;
            const int ri = ti * kTile + i, rj = tj * kTile + i;
            double av = 0.0, bv = 0.0;
            if (kr < k1) {
                const double ck = c ? c[kr] : 1.0;
                if (ri < p) av = u[(int64_t)ri * ldu + kr] * ck;
                if (rj < p) bv = u[(int64_t)rj * ldu + kr];
            }
            As[i][kk] = av;
            Bs[i][kk] = bv;
        }
        __syncthreads();
#pragma unroll 8
        for (int kk = 0; kk < kKc; ++kk) {
            double av[4], bv[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) av[a] = As[ty * 4 + a][kk];
#pragma unroll
            for (int bb = 0; bb < 4; ++bb) bv[bb] = Bs[tx * 4 + bb][kk];
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int bb = 0; bb < 4; ++bb) acc[a][bb] = fma(av[a], bv[bb], acc[a][bb]);
        }
        __syncthreads();
    }
    double *out = part + ((int64_t)s * npairs + pair) * (kTile * kTile);
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int bb = 0; bb < 4; ++bb) out[(ty * 4 + a) * kTile + tx * 4 + bb] = acc[a][bb];
}

// FP64 on the matrix cores (v_mfma_f64_16x16x4_f64), for p <= 512: per K chunk of kF64KC
// rows the workgroup stages every row of u once in LDS (FP64, as stored); its 8 waves own
// 16 x 16 blocks (bi <= bj) of the upper triangle in turn (block q of the workgroup's group
// to wave q mod 8) and run them from LDS, the A operand multiplied by c_k as it is read.  A
// group holds up to kF64Group blocks (p <= 256: all of them; beyond, the groups of one K range
// run on one XCD, see split_group).  An MFMA step takes 4 K values: lane l supplies
// A[bi*16 + l%16][k + l/16] and B[bj*16 + l%16][k + l/16] and holds D[l/16 + 4 r][l%16],
// r = 0..3, of its block (rows interleaved by 4).  The partials go to the 64 x 64 tile-pair
// layout of syrk_f64_kernel (blocks below the diagonal of a diagonal tile are never
// written, and syrk_reduce_kernel never reads them).
//
// Up to 256 columns the latency of a chunk's loads bounds it, then the matrix cores (100 columns:
// 36 us of their time for 200,000 rows).  So the next chunk is loaded while one is multiplied,
// and the kernel is built for several column counts: branches around absent row blocks and
// blocks, 17 + 2 x 16 of them per chunk whatever the count, cost more than the work at few
// columns.  A second LDS buffer (107 us against 93) and blocks without branches (138) did not
// pay.  Both products and their sums, 100,000 rows, before -> now, us: 10 columns 70 -> 31, 50: 102 -> 54,
// 150: 210 -> 161, 256: 455 -> 348.
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kF64Waves = 8, kF64KC = 32;
constexpr int kF64PerWave = 17, kF64Group = kF64Waves * kF64PerWave;   // 136 = all blocks at p <= 256

// MAXB: the most 16-row blocks, each with its own registers and LDS (32: p <= 512, 135 KB).
template <int MAXB>
__global__ __launch_bounds__(64 * kF64Waves, 1) void syrk_f64_mfma_kernel(const double *u, int64_t ldu, int p,
                                                                         const double *c, int64_t K,
                                                                         int64_t kchunk, double *part)
{
    constexpr bool kAhead = MAXB <= 16;
    // + 4: an operand, 16 rows x 4 columns, falls on all banks alike (beyond 256 columns + 1 measured the same)
    __shared__ double xs[MAXB * 16][kF64KC + (kAhead ? 4 : 1)];
    __shared__ double cs[kF64KC];
    // a wave's share of one group's blocks
    constexpr int kPW = MAXB <= 16 ? (MAXB * (MAXB + 1) / 2 + kF64Waves - 1) / kF64Waves : kF64PerWave;
    const int nb = (p + 15) / 16;
    const int nblk = nb * (nb + 1) / 2;
    const int nt = (p + kTile - 1) / kTile;
    const int npairs = nt * (nt + 1) / 2;
    const int lane = threadIdx.x & 63, w = kAhead ? __builtin_amdgcn_readfirstlane(threadIdx.x / 64) : (int)(threadIdx.x / 64);
    int s, grp;
    split_group(s, grp);
    const int q0 = grp * kF64Group;
    const int64_t k0 = (int64_t)s * kchunk;
    const int64_t k1 = k0 + kchunk < K ? k0 + kchunk : K;
    int bi[kPW], bj[kPW];
    f64x4 acc[kPW];
#pragma unroll
    for (int m = 0; m < kPW; ++m) {
        const int q = q0 + w + kF64Waves * m;
        int i = 0, rem = q < nblk ? q : 0;
        while (rem >= nb - i) {
            rem -= nb - i;
            ++i;
        }
        bi[m] = i;
        bj[m] = i + rem;
        acc[m] = f64x4{0.0, 0.0, 0.0, 0.0};
    }
    const int r16 = lane & 15, kq = lane >> 4;
    // This thread's entries of a chunk: column sk of rows sr, sr + 16, ...; columns beyond k1 count
    // as zero, rows beyond p as row p - 1 (their products are never read).  With up to 16 row
    // blocks the next chunk's are loaded while this one is multiplied, MAXB of them without a
    // branch around each; with more there are no registers for that.  Offsets from a uniform base take
    // 32 bits (ldu < 2^25).
    static_assert(64 * kF64Waves == 16 * kF64KC, "a pass of the workgroup stages 16 rows");
    const int sr = threadIdx.x / kF64KC, sk = threadIdx.x % kF64KC;
    const int srl = sr < p - 16 * (nb - 1) ? sr : p - 16 * (nb - 1) - 1;   // in the last row block
    double reg[kAhead ? MAXB : 1], creg = 1.0;
    auto load_chunk = [&](int64_t kc) {
        const int64_t left = k1 - 1 - kc;
        const uint32_t col = left < sk ? (uint32_t)left : (uint32_t)sk;
        const uint32_t at = (uint32_t)sr * (uint32_t)ldu + col, atl = (uint32_t)srl * (uint32_t)ldu + col;
        if constexpr (kAhead) {
#pragma unroll
            for (int m = 0; m < MAXB; ++m)
                reg[m] = (u + ((int64_t)16 * (m < nb ? m : nb - 1) * ldu + kc))[m >= nb - 1 ? atl : at];
        }
        if (c && threadIdx.x < kF64KC) creg = kc + sk < k1 ? c[kc + sk] : 1.0;
    };
    if (kAhead && k0 < k1) load_chunk(k0);
    for (int64_t kc = k0; kc < k1; kc += kF64KC) {
        if constexpr (kAhead) {
            const bool in = kc + sk < k1;
#pragma unroll
            for (int m = 0; m < MAXB; ++m) xs[16 * m + sr][sk] = in ? reg[m] : 0.0;
        } else {
            load_chunk(kc);
            for (int r = sr; r < nb * 16; r += 16)
                xs[r][sk] = (r < p && kc + sk < k1) ? u[(int64_t)r * ldu + kc + sk] : 0.0;
        }
        if (threadIdx.x < kF64KC) cs[threadIdx.x] = creg;
        __syncthreads();
        if (kAhead && kc + kF64KC < k1) load_chunk(kc + kF64KC);
#pragma unroll
        for (int ks = 0; ks < kF64KC; ks += 4) {
            const int kk = ks + kq;
            const double ck = cs[kk];
#pragma unroll
            for (int m = 0; m < kPW; ++m) {
                if (q0 + w + kF64Waves * m < nblk) {
                    const double a = xs[bi[m] * 16 + r16][kk] * ck;
                    const double b = xs[bj[m] * 16 + r16][kk];
                    acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[m], 0, 0, 0);
                }
            }
        }
        __syncthreads();   // the next chunk rewrites the staged rows
    }
#pragma unroll
    for (int m = 0; m < kPW; ++m) {
        if (q0 + w + kF64Waves * m < nblk) {
            const int ti = bi[m] / 4, tj = bj[m] / 4;
            const int pair = ti * nt - ti * (ti - 1) / 2 + (tj - ti);
            double *out = part + ((int64_t)s * npairs + pair) * (kTile * kTile);
            const int col = (bj[m] % 4) * 16 + r16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = (bi[m] % 4) * 16 + kq + 4 * r;
                out[row * kTile + col] = acc[m][r];
            }
        }
    }
}

// C (p x p, row-major, symmetric) = sign * sum over splits of the partial tiles, added to C
// when accumulate != 0.  Grid (npairs, 64): a workgroup takes 64 entries of one 64 x 64 tile;
// its 16 waves sum the splits q = w, w + 16, ... in order and the 16 sums are added in wave
// order (a fixed order: results do not vary run to run).  Entries below the diagonal of a
// diagonal tile are neither read nor written.
constexpr int kRedWaves = 16;

__global__ __launch_bounds__(64 * kRedWaves) void syrk_reduce_kernel(const double *part, int p, int S, double sign,
                                                                     int accumulate, double *C)
{
    __shared__ double red[kRedWaves][64];
    const int nt = (p + kTile - 1) / kTile;
    const int npairs = nt * (nt + 1) / 2;
    const int pair = blockIdx.x;
    int ti, tj;
    tile_pair(pair, nt, ti, tj);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int e = blockIdx.y * 64 + lane;
    const int a = e / kTile, bb = e % kTile;
    const int i = ti * kTile + a, j = tj * kTile + bb;
    const bool live = i < p && j < p && !(ti == tj && j < i);
    double s = 0.0;
    if (live)
        for (int q = w; q < S; q += kRedWaves) s += part[((int64_t)q * npairs + pair) * (kTile * kTile) + e];
    red[w][lane] = s;
    __syncthreads();
    if (w != 0 || !live) return;
    s = red[0][lane];
    for (int v = 1; v < kRedWaves; ++v) s += red[v][lane];
    s *= sign;
    if (accumulate) {
        C[(int64_t)i * p + j] += s;
        if (i != j) C[(int64_t)j * p + i] += s;
    } else {
        C[(int64_t)i * p + j] = s;
        if (i != j) C[(int64_t)j * p + i] = s;
    }
}

// Newton step: A (p x p, symmetric, restricted to the free columns: the others become unit
// rows) is factored as U'U unless `factored`, U overwriting A's upper triangle; then
// dx = -A^{-1} g on the free columns, 0 on the others.  status[0] = 1 if a pivot was not
// positive (that pivot is stored as -1).
//
// A single chain of p pivots bounds it, and around it the accesses between dependent steps.
// Up to kCholTail columns the packed triangle stays in one workgroup's LDS: 16-column panels, a
// wave factoring the diagonal block in registers, a thread per column for the rows to its
// right, and the rest updated by v_mfma_f64_16x16x4_f64 while the first wave already factors
// the next diagonal block.  Larger matrices are cut down to that by 64-column panels, two
// launches each over all tiles of what is left.  Before (one workgroup on global memory, a
// division per pivot and per solve step; beyond 512 columns unblocked) -> now, us by events:
// p = 20: 29 -> 18, 64: 77 -> 32, 200: 312 -> 120 (78 of it the factor, 26 the solves), 500:
// 1642 -> 403, 1000: 306,000 -> 1005.
constexpr int kCholTail = 200;   // 8 * (200 * 201 / 2 + 16 + 200) bytes of the 160 KB
constexpr int kPan = 16, kBlk = 64;

__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 1 / sqrt(d) and sqrt(d) to about an ulp for every d > 0: the hardware estimate, two Newton
// steps, and one for the root (a division and a root are several times as long a chain).  The steps go
// by d y, about sqrt(d), which neither overflows nor underflows where d itself does not.
__device__ __forceinline__ void pivot_root(double d, double &root, double &inv)
{
    d = fmin(d, 0x1.fffffffffffffp+1023);   // an overflowed diagonal takes its row and column out
    double y = __builtin_amdgcn_rsq(d);
    y = fma(0.5 * y, fma(-(d * y), y, 1.0), y);
    y = fma(0.5 * y, fma(-(d * y), y, 1.0), y);
    const double r = d * y;
    root = fma(0.5 * y, fma(-r, r, d), r);
    inv = y;
}

// An index that the compiler does not follow from one phase to the next: it would keep every
// address of every phase in a register of its own.
__device__ __forceinline__ int opaque(int x)
{
    asm volatile("" : "+s"(x));
    return x;
}

// Element (j, i), i >= j, of a packed upper triangle of order n: (j + 1, i) is n - 1 - j on.
__device__ __forceinline__ int tri(int j, int i, int n) { return j * n - j * (j + 1) / 2 + i; }

// The diagonal block at c0 (nb <= 16 columns) of the packed triangle T, by one wave: lane i
// holds column c0 + i.  Entries below the diagonal or beyond nb hold whatever is there (reads stay
// within kTriPad doubles of the triangle): nothing that is stored depends on them.
constexpr int kTriPad = 16;

__device__ __forceinline__ void factor_diagonal(double *T, int n, int c0, double *s_inv)
{
    const int lane = threadIdx.x & (kWaveC - 1), l16 = lane < kPan ? lane : kPan - 1;
    c0 = opaque(c0);
    const int nb = n - c0 < kPan ? n - c0 : kPan;
    double D[kPan];
    {
        int at = tri(c0, c0 + l16, n);
#pragma unroll
        for (int c = 0; c < kPan; at += c + 1 < nb ? n - 1 - c0 - c : 0, ++c) D[c] = T[at];
    }
#pragma unroll
    for (int k = 0; k < kPan; ++k) {
        const double d = lane_value(D[k], k);
        double root, inv;
        pivot_root(d, root, inv);
        if (!(d > 0.0)) root = -1.0;   // what is computed from here on is not used
        if (lane == 0) s_inv[k] = inv;
        D[k] = lane == k ? root : D[k] * inv;
#pragma unroll
        for (int q = k + 1; q < kPan; ++q) {
            D[q] = fma(-D[k], lane_value(D[k], q), D[q]);
            asm volatile("" : "+v"(D[q]));   // now: put off, the steps' rows would not fit in scalar registers
        }
    }
    int at = tri(opaque(c0), c0 + lane, n);
    const int last = lane < nb ? lane : -1;
#pragma unroll
    for (int c = 0; c < kPan; at += n - 1 - c0 - c, ++c)
        if (c <= last) T[at] = D[c];
}

// The packed triangle T (order n, in LDS, complete before the call) becomes its factor.
__device__ __forceinline__ void factor_packed(double *T, int n, double *s_inv)
{
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t / kWaveC), lane = t & (kWaveC - 1), waves = blockDim.x / kWaveC;
    const int r16 = lane & 15, kq = lane >> 4;
    for (int r0 = 0;; r0 += kPan) {
        if (r0 > 0) {
            const int c0 = r0 - kPan;
            // the panel's rows right of the block: U11' x = a, a column per thread
            for (int i = r0 + t; i < n; i += blockDim.x) {
                double a[kPan];
                const int cc = opaque(c0);
                int at = tri(cc, i, n);
#pragma unroll
                for (int c = 0; c < kPan; at += n - 1 - cc - c, ++c) a[c] = T[at];
                const double *row = T + tri(cc, cc, n);   // row[q]: entry (c0 + c, c0 + q)
#pragma unroll
                for (int c = 0; c < kPan; row += n - 1 - cc - c, ++c) {
                    a[c] *= s_inv[c];
#pragma unroll
                    for (int q = c + 1; q < kPan; ++q) a[q] = fma(-row[q], a[c], a[q]);
                    if (c % 4 == 3) asm volatile("" ::: "memory");   // all rows' reads would not fit in registers
                }
                at = tri(opaque(cc), i, n);
#pragma unroll
                for (int c = 0; c < kPan; at += n - 1 - cc - c, ++c) T[at] = a[c];
            }
            __syncthreads();
        }
        // A22 -= U12' U12 in 16 x 16 tiles; operands beyond n belong to results that are not stored
        const int nt = (n - r0 + kPan - 1) / kPan;
        auto tile = [&](int bi, int bj) {
            const int rb = opaque(r0), ri = rb + bi * kPan, rj = rb + bj * kPan;
            f64x4 acc;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = ri + kq + 4 * r, col = rj + r16;
                acc[r] = (col < n && row <= col) ? T[tri(row, col, n)] : 0.0;
            }
#pragma unroll
            for (int ks = 0; ks < kPan; ks += 4) {
                const int k = rb - kPan + ks + kq;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-T[tri(k, ri + r16, n)], T[tri(k, rj + r16, n)], acc, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = ri + kq + 4 * r, col = rj + r16;
                if (col < n && row <= col) T[tri(row, col, n)] = acc[r];
            }
        };
        if (w == 0) {
            if (r0 > 0) {
                tile(0, 0);
                wave_order();
            }
            factor_diagonal(T, n, r0, s_inv);
        } else if (r0 > 0) {
            for (int q = w; q < nt * (nt + 1) / 2; q += waves - 1) {   // tile 0 is the first wave's
                int i = 0, rem = q;
                while (rem >= nt - i) {
                    rem -= nt - i;
                    ++i;
                }
                tile(i, i + rem);
            }
        }
        __syncthreads();
        if (r0 + kPan >= n) return;
    }
}

// Rows and columns [r0, p) of A, p - r0 <= kCholTail: factored in LDS.  With r0 = 0 the step is
// solved as well (from A's stored factor if `factored`).  blockDim: at least 256 threads.
constexpr int kTailRows = 9;     // rows in flight per wave: 8 waves load 200 rows in three rounds
constexpr int kTailThreads = 512;   // more waves would leave too few registers (the diagonal block, the rows in flight)

__global__ __launch_bounds__(kTailThreads) void chol_tail_kernel(double *A, int p, int r0, const double *g,
                                                         const uint8_t *free_col, int factored, double *dx, int *status)
{
    extern __shared__ double T[];   // the packed triangle, kTriPad doubles, y [n] (r0 = 0)
    __shared__ double s_inv[kPan];
    __shared__ int s_bad;
    const int n = p - r0;
    double *y = T + n * (n + 1) / 2 + kTriPad;
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t / kWaveC), lane = t & (kWaveC - 1), waves = blockDim.x / kWaveC;
    const bool mask = r0 == 0 && !factored;   // larger matrices were masked by their first launch
    constexpr int kQ = (kCholTail + kWaveC - 1) / kWaveC;
    int fi[kQ];   // of column 64 q + lane
    for (int j0 = w; j0 < n; j0 += kTailRows * waves) {
        double v[kTailRows][kQ];
#pragma unroll
        for (int m = 0; m < kTailRows; ++m) {
            const int j = j0 + m * waves < n ? j0 + m * waves : n - 1;
            const double *row = A + (int64_t)(r0 + j) * p + r0;
#pragma unroll
            for (int q = 0; q < kQ; ++q) {
                const int i = q * kWaveC + lane;
                v[m][q] = 0.0;
                if (q * kWaveC < n && (q + 1) * kWaveC > j) v[m][q] = row[i < n ? i : n - 1];
            }
        }
        if (j0 == w) {
#pragma unroll
            for (int q = 0; q < kQ; ++q) {
                const int i = q * kWaveC + lane;
                fi[q] = mask ? free_col[i < n ? i : n - 1] : 1;
            }
            if (t == 0) s_bad = 0;
            if (t < kTriPad) T[n * (n + 1) / 2 + t] = 0.0;
            if (r0 == 0)
                for (int i = t; i < n; i += blockDim.x) y[i] = free_col[i] ? -g[i] : 0.0;
        }
#pragma unroll
        for (int m = 0; m < kTailRows; ++m) {
            const int j = j0 + m * waves;
            const int fl = j < kWaveC ? fi[0] : j < 2 * kWaveC ? fi[1] : j < 3 * kWaveC ? fi[2] : fi[kQ - 1];
            const int fj = __builtin_amdgcn_readlane(fl, j & (kWaveC - 1));
#pragma unroll
            for (int q = 0; q < kQ; ++q) {
                const int i = q * kWaveC + lane;
                if (j < n && i >= j && i < n) T[tri(j, i, n)] = (fj && fi[q]) ? v[m][q] : (i == j ? 1.0 : 0.0);
            }
        }
    }
    static_assert(kQ == 4, "the row's own flag is taken from one of four registers");
    __syncthreads();
    if (!factored) {
        factor_packed(T, n, s_inv);
        for (int j = w; j < n; j += waves)
            for (int i = j + lane; i < n; i += kWaveC) A[(int64_t)(r0 + j) * p + r0 + i] = T[tri(j, i, n)];
    }
    if (r0 != 0) return;
    __syncthreads();
    // the diagonal becomes its inverse
    for (int i = t; i < n; i += blockDim.x) {
        const double d = T[tri(i, i, n)];
        if (!(d > 0.0)) s_bad = 1;
        T[tri(i, i, n)] = 1.0 / d;
    }
    __syncthreads();
    // U' y = -g, then U x = y: 64 unknowns by one wave (an unknown per lane), the others by all
    for (int k0 = 0; k0 < n; k0 += kBlk) {
        const int nb = n - k0 < kBlk ? n - k0 : kBlk;
        if (w == 0) {
            const int i = k0 + lane;
            double yi = lane < nb ? y[i] : 0.0;
            const double inv = lane < nb ? T[tri(i, i, n)] : 0.0;
            int at = tri(k0, i < n ? i : n - 1, n);
            for (int c0 = 0; c0 < nb; c0 += kPan) {
                double u[kPan];   // rows beyond nb: the last one again, times y = 0
#pragma unroll
                for (int c = 0; c < kPan; at += c0 + c + 1 < nb ? n - 1 - k0 - c0 - c : 0, ++c) u[c] = T[at];
#pragma unroll
                for (int c = 0; c < kPan; ++c) {
                    const double yc = lane_value(yi * inv, c0 + c);
                    yi = fma(lane > c0 + c ? -u[c] : 0.0, yc, yi);
                }
            }
            if (lane < nb) y[i] = yi * inv;
        }
        __syncthreads();
        for (int i = k0 + nb + t; i < n; i += blockDim.x) {
            double acc = y[i];
#pragma unroll 16
            for (int c = 0; c < nb; ++c) acc = fma(-T[tri(k0 + c, i, n)], y[k0 + c], acc);
            y[i] = acc;
        }
        __syncthreads();
    }
    for (int k0 = (n - 1) / kBlk * kBlk; k0 >= 0; k0 -= kBlk) {
        const int nb = n - k0 < kBlk ? n - k0 : kBlk;
        if (w == 0) {
            const int i = k0 + lane;
            double xi = lane < nb ? y[i] : 0.0;
            const double inv = lane < nb ? T[tri(i, i, n)] : 0.0;
            const double *row = T + tri(i < n ? i : n - 1, k0, n);
            for (int c0 = (nb - 1) / kPan * kPan; c0 >= 0; c0 -= kPan) {
                double u[kPan];   // at most kTriPad - 1 entries beyond the triangle
#pragma unroll
                for (int c = 0; c < kPan; ++c) u[c] = row[c0 + c];
#pragma unroll
                for (int c = kPan - 1; c >= 0; --c) {
                    const double xc = lane_value(xi * inv, c0 + c);
                    xi = fma(lane < c0 + c && c0 + c < nb ? -u[c] : 0.0, xc, xi);
                }
            }
            if (lane < nb) y[i] = xi * inv;
        }
        __syncthreads();
        for (int i = t; i < k0; i += blockDim.x) {
            double acc = y[i];
            const double *row = T + tri(i, k0, n);
#pragma unroll 16
            for (int c = 0; c < nb; ++c) acc = fma(-row[c], y[k0 + c], acc);
            y[i] = acc;
        }
        __syncthreads();
    }
    for (int i = t; i < n; i += blockDim.x) dx[i] = free_col[i] ? y[i] : 0.0;
    if (t == 0) status[0] = s_bad;
}

// One 64 x 64 tile (bi <= bj) of what is left from column r0 on: the first launch (c0 < 0) makes
// the rows and columns that are not free unit rows, the later ones subtract the panel of rows
// [c0, c0 + 64) = [r0 - 64, r0).  The first tile's workgroup goes on to factor it when another
// panel follows.  Grid: the tiles; 256 threads.
__global__ __launch_bounds__(256) void chol_tile_kernel(double *A, int p, int c0, int r0, const uint8_t *free_col,
                                                        int panel_follows)
{
    __shared__ double ui[kBlk][kBlk + 1], uj[kBlk][kBlk + 1];
    __shared__ double s_inv[kPan];
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t / kWaveC), lane = t & (kWaveC - 1);
    const int r16 = lane & 15, kq = lane >> 4;
    const int nt = (p - r0 + kBlk - 1) / kBlk;
    int bi = 0, rem = blockIdx.x;
    while (rem >= nt - bi) {
        rem -= nt - bi;
        ++bi;
    }
    const int ri = r0 + bi * kBlk, rj = r0 + (bi + rem) * kBlk;
    if (c0 >= 0) {
        double vi[kBlk / 4], vj[kBlk / 4];
#pragma unroll
        for (int m = 0; m < kBlk / 4; ++m) {
            const double *row = A + (int64_t)(c0 + w + 4 * m) * p;
            vi[m] = ri + lane < p ? row[ri + lane] : 0.0;
            vj[m] = rj + lane < p ? row[rj + lane] : 0.0;
        }
#pragma unroll
        for (int m = 0; m < kBlk / 4; ++m) {
            ui[w + 4 * m][lane] = vi[m];
            uj[w + 4 * m][lane] = vj[m];
        }
        __syncthreads();
    }
    // wave w: rows 16 w .. 16 w + 15 of the tile
    f64x4 acc[4];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = ri + w * kPan + kq + 4 * r, col = rj + b * kPan + r16;
            acc[b][r] = 0.0;
            if (col < p && row <= col) {
                acc[b][r] = A[(int64_t)row * p + col];
                if (c0 < 0 && !(free_col[row] && free_col[col])) acc[b][r] = row == col ? 1.0 : 0.0;
            }
        }
    if (c0 >= 0) {
#pragma unroll 4
        for (int ks = 0; ks < kBlk; ks += 4) {
            const double a = -ui[ks + kq][w * kPan + r16];
#pragma unroll
            for (int b = 0; b < 4; ++b)
                acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, uj[ks + kq][b * kPan + r16], acc[b], 0, 0, 0);
        }
        __syncthreads();
    }
    const bool factor = blockIdx.x == 0 && panel_follows;   // ri = rj = r0 and r0 + 64 < p
    double *T = &ui[0][0];   // packed, order 64
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = ri + w * kPan + kq + 4 * r, col = rj + b * kPan + r16;
            if (col < p && row <= col) {
                if (factor) T[tri(row - r0, col - r0, kBlk)] = acc[b][r];
                else A[(int64_t)row * p + col] = acc[b][r];
            }
        }
    if (!factor) return;
    __syncthreads();
    factor_packed(T, kBlk, s_inv);
    for (int j = w; j < kBlk; j += 4)
        if (lane >= j) A[(int64_t)(r0 + j) * p + r0 + lane] = T[tri(j, lane, kBlk)];
}

// The rows [c0, c0 + 64) right of their factored diagonal block: U11' X = A12, 64 columns per workgroup
// of 256 threads.
__global__ __launch_bounds__(256) void chol_rows_kernel(double *A, int p, int c0)
{
    __shared__ double U[kBlk][kBlk + 1], X[kBlk][kBlk + 1];
    __shared__ double s_inv[kBlk];
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t / kWaveC), lane = t & (kWaveC - 1);
    const int r16 = lane & 15, kq = lane >> 4;
    const int col = c0 + kBlk + blockIdx.x * kBlk + lane;
    double vu[kBlk / 4], vx[kBlk / 4];
#pragma unroll
    for (int m = 0; m < kBlk / 4; ++m) {
        const double *row = A + (int64_t)(c0 + w + 4 * m) * p;
        vu[m] = lane >= w + 4 * m ? row[c0 + lane] : 0.0;
        vx[m] = col < p ? row[col] : 0.0;
    }
#pragma unroll
    for (int m = 0; m < kBlk / 4; ++m) {
        const int j = w + 4 * m;
        U[j][lane] = vu[m];
        X[j][lane] = vx[m];
        if (lane == j) s_inv[j] = vu[m] > 0.0 ? 1.0 / vu[m] : 1.0;
    }
    __syncthreads();
    for (int b0 = 0; b0 < kBlk; b0 += kPan) {
        if (w == 0) {
            double a[kPan];
#pragma unroll
            for (int c = 0; c < kPan; ++c) a[c] = X[b0 + c][lane];
#pragma unroll
            for (int c = 0; c < kPan; ++c) {
                a[c] *= s_inv[b0 + c];
#pragma unroll
                for (int q = c + 1; q < kPan; ++q) a[q] = fma(-U[b0 + c][b0 + q], a[c], a[q]);
                if (c % 4 == 3) asm volatile("" ::: "memory");
            }
#pragma unroll
            for (int c = 0; c < kPan; ++c) X[b0 + c][lane] = a[c];
        }
        __syncthreads();
        // the rows below, wave w the 16 columns from 16 w on
        for (int rb = b0 + kPan; rb < kBlk; rb += kPan) {
            f64x4 acc;
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = X[rb + kq + 4 * r][w * kPan + r16];
#pragma unroll
            for (int ks = 0; ks < kPan; ks += 4)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-U[b0 + ks + kq][rb + r16], X[b0 + ks + kq][w * kPan + r16],
                                                           acc, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) X[rb + kq + 4 * r][w * kPan + r16] = acc[r];
        }
        __syncthreads();
    }
    if (col < p)
#pragma unroll
        for (int m = 0; m < kBlk / 4; ++m) A[(int64_t)(c0 + w + 4 * m) * p + col] = X[w + 4 * m][lane];
}

// U'U x = -g from the stored factor, for p > kCholTail: blocks of 64 unknowns, their diagonal
// block staged in LDS (the next one loaded while the others are updated).
constexpr int kSolveThreads = 1024;

__global__ __launch_bounds__(kSolveThreads) void chol_solve_kernel(const double *A, int p, const double *g,
                                                                   const uint8_t *free_col, double *dx, int *status)
{
    extern __shared__ double y[];   // [p]
    __shared__ double U[kBlk][kBlk + 1];
    __shared__ int s_bad;
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t / kWaveC), lane = t & (kWaveC - 1);
    constexpr int kWaves = kSolveThreads / kWaveC, kM = kBlk / kWaves;
    static_assert(kBlk == kWaveC && kBlk % kWaves == 0, "a wave stages whole rows");
    if (t == 0) s_bad = 0;
    for (int i = t; i < p; i += kSolveThreads) y[i] = free_col[i] ? -g[i] : 0.0;
    double v[kM];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int m = 0; m < kM; ++m) {
            const int j = w + kWaves * m;
            v[m] = (k0 >= 0 && k0 + lane < p && lane >= j) ? A[(int64_t)(k0 + j) * p + k0 + lane] : (lane == j ? 1.0 : 0.0);
        }
    };
    auto stage = [&]() {   // the diagonal as its inverse
#pragma unroll
        for (int m = 0; m < kM; ++m) {
            const int j = w + kWaves * m;
            if (lane == j && !(v[m] > 0.0)) s_bad = 1;
            U[j][lane] = lane == j ? 1.0 / v[m] : v[m];
        }
    };
    __syncthreads();
    fetch(0);
    for (int k0 = 0; k0 < p; k0 += kBlk) {
        stage();
        __syncthreads();
        fetch(k0 + kBlk < p ? k0 + kBlk : k0);   // the last block is the next solve's first
        const int nb = p - k0 < kBlk ? p - k0 : kBlk;
        if (w == 0) {
            double yi = lane < nb ? y[k0 + lane] : 0.0;
            const double inv = U[lane][lane];
#pragma unroll 16
            for (int c = 0; c < kBlk; ++c) {
                const double u = U[c][lane];
                yi = fma(lane > c ? -u : 0.0, lane_value(yi * inv, c), yi);
            }
            if (lane < nb) y[k0 + lane] = yi * inv;
        }
        __syncthreads();
        // 64 columns per wave
        for (int i = k0 + kBlk + t; i < p; i += kSolveThreads) {
            double acc = y[i];
#pragma unroll 16
            for (int c = 0; c < kBlk; ++c) acc = fma(-A[(int64_t)(k0 + c) * p + i], y[k0 + c], acc);
            y[i] = acc;
        }
    }
    for (int k0 = (p - 1) / kBlk * kBlk; k0 >= 0; k0 -= kBlk) {
        __syncthreads();
        stage();
        __syncthreads();
        fetch(k0 - kBlk);
        const int nb = p - k0 < kBlk ? p - k0 : kBlk;
        if (w == 0) {
            double xi = lane < nb ? y[k0 + lane] : 0.0;
            const double inv = U[lane][lane];
#pragma unroll 16
            for (int c = kBlk - 1; c >= 0; --c) {
                const double u = U[lane][c];
                xi = fma(lane < c ? -u : 0.0, lane_value(xi * inv, c), xi);
            }
            if (lane < nb) y[k0 + lane] = xi * inv;
        }
        __syncthreads();
        // a row per wave, a column per lane
        const double xc = lane < nb ? y[k0 + lane] : 0.0;
#pragma unroll 4
        for (int i = w; i < k0; i += kWaves) {
            double acc = lane < nb ? A[(int64_t)i * p + k0 + lane] * xc : 0.0;
#pragma unroll
            for (int o = kWaveC / 2; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, kWaveC);
            if (lane == 0) y[i] -= acc;
        }
    }
    __syncthreads();
    for (int i = t; i < p; i += kSolveThreads) dx[i] = free_col[i] ? y[i] : 0.0;
    if (t == 0) status[0] = s_bad;
}

// ------------------------------------------------------------------ BF16 on the matrix cores

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4v __attribute__((ext_vector_type(4)));

constexpr int kMT = 32;              // MFMA tile edge
constexpr int kTilesPerWave = 8;
constexpr int kSyrkBfWaves = 4;
constexpr int kPairsPerGroup = kTilesPerWave * kSyrkBfWaves;

__host__ __device__ __forceinline__ int npairs32(int p)
{
    const int nt = (p + kMT - 1) / kMT;
    return nt * (nt + 1) / 2;
}

// LDS-staged variant for p <= 256 (at most 8 row tiles): per 64-row K chunk
// the workgroup stages all row tiles of u once (and once more multiplied by
// the weights, rounded to BF16), then every wave runs its tile pairs' MFMAs
// from LDS.  The next chunk's global loads are issued into registers before
// the current chunk's MFMAs.  part[(s * npairs + pair) * 1024 + m * 32 + n] = sum over K range s of
// c_k u[ti*32+m][k] u[tj*32+n][k] (scaled units).  Grid (S, pair groups).
// BLK: u is [ldu / 8][p][8], a thread's pieces are one K unit of rows 64 apart, not K units of a row.

// MAXT: the most row tiles the launch may have (the LDS holds MAXT x 32 rows); OCC: the waves
// per SIMD the register budget is cut for (with NWV waves of TPW tile pairs each: two
// workgroups of 8 waves per compute unit need 4, so one workgroup's loads overlap the
// other's matrix-core work).
template <bool WEIGHT, bool BLK, int KC, int MAXT, int OCC, int NWV, int TPW>
__global__ __launch_bounds__(64 * NWV, OCC) void syrk_bf16_lds_kernel(const uint16_t *u, int64_t ldu, int p,
                                                                               const double *c, int64_t K,
                                                                               int64_t kchunk, float *part)
{
    constexpr int kLdsKC = KC, kLdsStride = KC + 8, kLdsPieces = KC / 8;
    static_assert(NWV * TPW == kPairsPerGroup, "a group holds kPairsPerGroup tile pairs");
    static_assert(!BLK || NWV == kLdsPieces, "a wave stages one K unit of the chunk");
    constexpr int kLdsPerThread = (MAXT * kMT * kLdsPieces + 64 * NWV - 1) / (64 * NWV);
    extern __shared__ uint16_t sh[];   // [nt*32][kLdsStride] plain, then weighted (WEIGHT)
    __shared__ float cw[kLdsKC];
    const int nt = (p + kMT - 1) / kMT;
    const int rows = nt * kMT;
    uint16_t *plain = sh;
    uint16_t *wtd = sh + (size_t)rows * kLdsStride;
    const int npairs = nt * (nt + 1) / 2;
    const int lane = threadIdx.x & 63, w = threadIdx.x / 64;
    int s, grp;
    split_group(s, grp);
    const int pair0 = grp * kPairsPerGroup + w * TPW;
    const int nq = npairs - pair0 < TPW ? (npairs - pair0 > 0 ? npairs - pair0 : 0) : TPW;
    const int64_t k0 = (int64_t)s * kchunk;
    const int64_t k1 = k0 + kchunk < K ? k0 + kchunk : K;
    const int rsub = lane & 31, ksub = 8 * (lane >> 5);
    // LDS offsets of this lane's A (weighted) and B (plain) rows for each tile pair, packed
    // 16 bits each (at most 8 x 32 rows of kLdsStride elements: < 2^16)
    uint32_t offs[TPW];
    f32x16 acc[TPW];
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
        int ti, tj;
        tile_pair(pair0 + q < npairs ? pair0 + q : 0, nt, ti, tj);
        offs[q] = (uint32_t)((ti * kMT + rsub) * kLdsStride) | ((uint32_t)((tj * kMT + rsub) * kLdsStride) << 16);
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[q][i] = 0.0f;
    }
    // prefetch registers: this thread's pieces, one chunk ahead
    u32x4v reg[kLdsPerThread];
    float creg = 0.0f;
    auto load_chunk = [&](int64_t kc) {
#pragma unroll
        for (int m = 0; m < kLdsPerThread; ++m) {
            const int e = threadIdx.x + 64 * NWV * m;
            const int r = BLK ? lane + 64 * m : e / kLdsPieces, piece = BLK ? w : e % kLdsPieces;
            u32x4v v = {0u, 0u, 0u, 0u};
            if (r < p)
                v = *reinterpret_cast<const u32x4v *>(BLK ? u + ((kc / 8 + piece) * p + r) * 8
                                                          : u + (int64_t)r * ldu + kc + 8 * piece);
            reg[m] = v;
        }
        if (WEIGHT && threadIdx.x < kLdsKC) creg = (float)c[kc + threadIdx.x];
    };
    if (k0 < k1) load_chunk(k0);
    for (int64_t kc = k0; kc < k1; kc += kLdsKC) {
        if (WEIGHT && threadIdx.x < kLdsKC) cw[threadIdx.x] = creg;
        __syncthreads();
#pragma unroll
        for (int m = 0; m < kLdsPerThread; ++m) {
            const int e = threadIdx.x + 64 * NWV * m;
            const int r = BLK ? lane + 64 * m : e / kLdsPieces, piece = BLK ? w : e % kLdsPieces;
            if (r < rows) {
                *reinterpret_cast<u32x4v *>(plain + r * kLdsStride + 8 * piece) = reg[m];
                if (WEIGHT) {
                    const bf16x8 x = __builtin_bit_cast(bf16x8, reg[m]);
                    bf16x8 y;
#pragma unroll
                    for (int i = 0; i < 8; ++i) y[i] = (__bf16)((float)x[i] * cw[8 * piece + i]);
                    *reinterpret_cast<u32x4v *>(wtd + r * kLdsStride + 8 * piece) = __builtin_bit_cast(u32x4v, y);
                }
            }
        }
        __syncthreads();
        if (kc + kLdsKC < k1) load_chunk(kc + kLdsKC);   // in flight during the MFMAs below
        const uint16_t *asrc = WEIGHT ? wtd : plain;
#pragma unroll
        for (int sub = 0; sub < kLdsKC / 16; ++sub) {
            const int kk = 16 * sub + ksub;
            // a wave's pairs run along rows of the upper triangle: the A fragment (row tile ti)
            // is read from LDS only when ti changes
            bf16x8 a;
#pragma unroll
            for (int q = 0; q < TPW; ++q) {
                if (q < nq) {
                    if (q == 0 || (offs[q] & 0xffffu) != (offs[q - 1] & 0xffffu))
                        a = __builtin_bit_cast(bf16x8,
                                               *reinterpret_cast<const u32x4v *>(asrc + (offs[q] & 0xffffu) + kk));
                    const bf16x8 b = __builtin_bit_cast(
                        bf16x8, *reinterpret_cast<const u32x4v *>(plain + (offs[q] >> 16) + kk));
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[q], 0, 0, 0);
                }
            }
        }
        __syncthreads();   // the next chunk rewrites the LDS tiles
    }
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
        if (q < nq) {
            float *out = part + ((int64_t)s * npairs + pair0 + q) * (kMT * kMT);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int m = 8 * (i / 4) + 4 * (lane / 32) + (i % 4), n = lane % 32;
                out[m * kMT + n] = acc[q][i];
            }
        }
    }
}

// More than 8 row tiles: the tile pairs are cut into blocks of 8 x 8 (row block I, column block
// J >= I), one block and K range per workgroup of 8 waves.  Per 64-row chunk the rows of block I
// are staged in LDS multiplied by the weights (FP32, rounded to BF16) and those of block J as
// they are; two buffers and one barrier per chunk, the next chunk's loads in flight during the
// products.  Off the diagonal a wave holds 2 x 4 tiles, so 6 fragments read from LDS feed
// 8 products (a wave of 4 tile pairs in a row needs 5 for 4: the LDS, not the matrix cores, set
// the pace).  An element is staged once per
// block that it takes part in -- 5 times at p = 1000, where 4 x 4 blocks with both copies of
// every row staged it 9 times.  Measured: N = 1e6, p = 1000 with weights 4.50 -> 1.85 ms (0.55
// PFLOP/s of the upper triangle), half as many rows without 0.91 -> 0.66 ms; 1.25e6 rows, p = 500
// 1.11 -> 0.50 ms.  Same partial layout as the kernels above.
constexpr int kWideTiles = 8, kWideRows = kWideTiles * kMT, kWideWaves = 8, kWideKC = 64, kWideStride = kWideKC + 8;
constexpr int kWidePer = kWideRows * (kWideKC / 8) / (64 * kWideWaves);   // 16-byte pieces per thread and operand: 4

__host__ __device__ __forceinline__ int pair_index(int ti, int tj, int nt)
{
    return ti * nt - ti * (ti - 1) / 2 + (tj - ti);   // row-major upper triangle, ti <= tj
}

__device__ __forceinline__ void store_tile(float *part, int64_t slot, const f32x16 &acc, int lane)
{
    float *out = part + slot * (kMT * kMT);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int m = 8 * (i / 4) + 4 * (lane / 32) + (i % 4), n = lane % 32;
        out[m * kMT + n] = acc[i];
    }
}

// Wave w's 2 x 4 tiles of a block: rows 2 wr.., columns 4 wc..; returns the mask of the wanted ones.
// On the diagonal the eight regions hold 8, 8, 7, 7, 3, 3, 0 and 0 wanted tiles (row <= column),
// dealt so that the two waves of a SIMD (w, w + 4) have 8, 8, 10 and 10.
__device__ __forceinline__ uint32_t wide_region(int w, bool diag, int &wr, int &wc)
{
    wr = diag ? (0x31322010 >> (4 * w)) & 3 : w / 2;
    wc = diag ? (0x10001011 >> (4 * w)) & 1 : w % 2;
    uint32_t want = 0xffu;
    if (diag) {
        want = 0u;
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (2 * wr + q / 4 <= 4 * wc + q % 4) want |= 1u << q;
    }
    return __builtin_amdgcn_readfirstlane(want);
}

template <bool WEIGHT, bool BLK>
__global__ __launch_bounds__(64 * kWideWaves, 2) void syrk_bf16_wide_kernel(const uint16_t *u, int64_t ldu, int p,
                                                                           const double *c, int64_t K, int64_t kchunk,
                                                                           float *part)
{
    extern __shared__ uint16_t sh[];   // two buffers of [A rows, B rows][kWideStride]
    constexpr int kHalf = kWideRows * kWideStride;
    const int nt = (p + kMT - 1) / kMT;
    const int nb = (nt + kWideTiles - 1) / kWideTiles;
    const int npairs = nt * (nt + 1) / 2;
    int I, J, s, grp;
    split_group(s, grp);
    tile_pair(grp, nb, I, J);
    const bool diag = I == J;
    const bool both = !diag || WEIGHT;   // a diagonal block without weights reads one copy twice
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t / 64);
    const int64_t k0 = (int64_t)s * kchunk;
    const int64_t k1 = k0 + kchunk < K ? k0 + kchunk : K;
    // this thread's rows: row + 64 m (BLK: u is [ldu / 8][p][8], consecutive rows of a K unit lie together)
    const int piece = BLK ? w : t % 8, row = BLK ? lane : t / 8;
    u32x4v ra[kWidePer], rb[kWidePer];
    float wt[8];
    auto load = [&](int64_t kc) {
#pragma unroll
        for (int m = 0; m < kWidePer; ++m) {
            const int i = I * kWideRows + row + 64 * m, j = J * kWideRows + row + 64 * m;
            u32x4v va = {0u, 0u, 0u, 0u}, vb = {0u, 0u, 0u, 0u};
            auto at = [&](int r) {
                return reinterpret_cast<const u32x4v *>(BLK ? u + ((kc / 8 + piece) * p + r) * 8
                                                            : u + (int64_t)r * ldu + kc + 8 * piece);
            };
            if (i < p) va = *at(i);
            if (!diag && j < p) vb = *at(j);
            ra[m] = va;
            rb[m] = vb;
        }
        if constexpr (WEIGHT) {
#pragma unroll
            for (int i = 0; i < 8; ++i) wt[i] = (float)c[kc + 8 * piece + i];
        }
    };
    auto stage = [&](int buf) {
        uint16_t *pa = sh + buf * 2 * kHalf + row * kWideStride + 8 * piece, *pb = pa + kHalf;
#pragma unroll
        for (int m = 0; m < kWidePer; ++m) {
            u32x4v va = ra[m];
            if constexpr (WEIGHT) {
                const bf16x8 x = __builtin_bit_cast(bf16x8, va);
                bf16x8 y;
#pragma unroll
                for (int i = 0; i < 8; ++i) y[i] = (__bf16)((float)x[i] * wt[i]);
                va = __builtin_bit_cast(u32x4v, y);
            }
            *reinterpret_cast<u32x4v *>(pa + 64 * m * kWideStride) = va;
            if (both) *reinterpret_cast<u32x4v *>(pb + 64 * m * kWideStride) = diag ? ra[m] : rb[m];
        }
    };
    f32x16 acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[q][i] = 0.0f;
    // a fragment: row tile's row lane % 32, 8 K values from 8 (lane / 32)
    const int frag = (lane & 31) * kWideStride + 8 * (lane >> 5);
    int wr, wc;
    const uint32_t want = wide_region(w, diag, wr, wc);
    const uint16_t *fa = sh + 2 * wr * kMT * kWideStride + frag;
    const uint16_t *fb = sh + (both ? kHalf : 0) + 4 * wc * kMT * kWideStride + frag;
    auto products = [&](int buf) {
        const uint16_t *A = fa + buf * 2 * kHalf, *B = fb + buf * 2 * kHalf;
        auto get = [](const uint16_t *src) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4v *>(src)); };
        if (want == 0u) return;
#pragma unroll
        for (int k = 0; k < kWideKC; k += 16) {
            bf16x8 a[2], b[4];
#pragma unroll
            for (int i = 0; i < 2; ++i) a[i] = get(A + i * kMT * kWideStride + k);
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = get(B + j * kMT * kWideStride + k);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (want & (1u << (4 * i + j)))
                        acc[4 * i + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[4 * i + j], 0, 0, 0);
        }
    };
    if (k0 < k1) {
        load(k0);
        stage(0);
        if (k0 + kWideKC < k1) load(k0 + kWideKC);
    }
    __syncthreads();
    int buf = 0;
    for (int64_t kc = k0; kc < k1; kc += kWideKC, buf ^= 1) {
        products(buf);
        if (kc + kWideKC < k1) {
            stage(buf ^ 1);   // last read before the previous barrier
            if (kc + 2 * kWideKC < k1) load(kc + 2 * kWideKC);
        }
        __syncthreads();
    }
    const int64_t base = (int64_t)s * npairs;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int ti = I * kWideTiles + 2 * wr + q / 4, tj = J * kWideTiles + 4 * wc + q % 4;
        if ((want & (1u << q)) && ti < nt && tj < nt) store_tile(part, base + pair_index(ti, tj, nt), acc[q], lane);
    }
}

// ------------------------------------------------------------------ FP8 (e4m3) on the matrix cores
//
// X is stored as e4m3 with a power-of-two scale per column (|x / s| <= 224).
// For X' diag(b) X both operands are the same matrix a_rj = (x_rj / s_j)
// sqrt(b_r) / S, with S the power of two >= sqrt(max b): each 64-row K chunk
// of every row tile is read once, multiplied by sqrt(b_r)/S in FP32 and
// rounded to e4m3 into LDS, and the waves run v_mfma_scale_f32_32x32x64_f8f6f4
// (unit block scales) on their tile pairs.  The FP32 partials are summed in
// FP64 times s_i s_j S^2.

constexpr float kFp8Max = 224.0f;   // below the e4m3 maximum of either encoding
constexpr int kF8KC = 64, kF8Stride = 80;   // bytes per LDS row (64 + 16 pad)
// Most staged rows of the one-pass kernel (p rounded up to 32).  Up to 320 its two groups of tile pairs convert
// 640 rows per chunk, three blocks of 256 x 256 convert 1024 (N = 4e5, P = 257: 181 us against 218 with
// the product of Z, P = 320: 193 against 224); from a third group on the blocks win (P = 352: 292
// against 237).
constexpr int kF8Rows = 320;
typedef int i32x8v __attribute__((ext_vector_type(8)));

// The e4m3 copy is stored in blocks of kF8KC rows of X: block k holds, for each
// of the prow (= p rounded up to 32) columns in turn, its kF8KC bytes (zero for
// the padding columns), so the contraction reads each chunk as one contiguous
// stretch of prow * kF8KC bytes.
__global__ __launch_bounds__(256) void to_fp8_kernel(const double *x, int64_t ld, int p, int prow,
                                                     const float *xscale, uint8_t *x8)
{
    const int j = blockIdx.y;
    const int64_t r = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (r >= ld) return;
    int v = 0;
    if (j < p) {
        const double inv = 1.0 / (double)xscale[j];
        const double *src = x + (int64_t)j * ld + r;
        v = __builtin_amdgcn_cvt_pk_fp8_f32((float)(src[0] * inv), (float)(src[1] * inv), 0, false);
        v = __builtin_amdgcn_cvt_pk_fp8_f32((float)(src[2] * inv), (float)(src[3] * inv), v, true);
    }
    *reinterpret_cast<int *>(x8 + ((r / kF8KC) * prow + j) * kF8KC + r % kF8KC) = v;
}

// wsc[0] = S = 2^ceil(log2(sqrt(max b))) (1 if b is all zero), in two launches
__global__ __launch_bounds__(256) void bmax_kernel(const double *b, int64_t n, double *blockmax)
{
    __shared__ double red[4];
    double m = 0.0;
    for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < n; r += (int64_t)gridDim.x * 256) m = fmax(m, b[r]);
    for (int off = 32; off >= 1; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = m;
    __syncthreads();
    if (threadIdx.x == 0) blockmax[blockIdx.x] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

__global__ __launch_bounds__(256) void wscale_kernel(const double *blockmax, int nb, double *wsc)
{
    __shared__ double red[4];
    double m = 0.0;
    for (int i = threadIdx.x; i < nb; i += 256) m = fmax(m, blockmax[i]);
    for (int off = 32; off >= 1; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
        wsc[0] = m > 0.0 ? exp2(ceil(log2(sqrt(m)))) : 1.0;
    }
}

// Two waves per SIMD (registers capped at 256, accumulators included): the
// products of one chunk overlap the other wave's staging.
// NWV waves of TPW tile pairs each, registers cut for two workgroups per compute unit.
template <int NWV = kSyrkBfWaves, int TPW = kTilesPerWave>
__global__ __launch_bounds__(64 * NWV, NWV / 2) void syrk_fp8_lds_kernel(const uint8_t *u, int p,
                                                                        const double *c, const double *wsc,
                                                                        int64_t K, int64_t kchunk, float *part)
{
    extern __shared__ uint8_t sh8[];   // [nt*32][kF8Stride]
    __shared__ float cw[kF8KC];
    const int nt = (p + kMT - 1) / kMT;
    const int rows = nt * kMT;
    const int npairs = nt * (nt + 1) / 2;
    const int lane = threadIdx.x & 63, w = threadIdx.x / 64;
    int s, grp;
    split_group(s, grp);
    const int pair0 = grp * kPairsPerGroup + w * TPW;
    const int nq = npairs - pair0 < TPW ? (npairs - pair0 > 0 ? npairs - pair0 : 0) : TPW;
    const int64_t k0 = (int64_t)s * kchunk;
    const int64_t k1 = k0 + kchunk < K ? k0 + kchunk : K;
    const double invS = 1.0 / wsc[0];
    const int rsub = lane & 31, kofs = 32 * (lane >> 5);
    // LDS byte offsets of this lane's A and B rows for each tile pair, packed 16 bits each
    // (at most kF8Rows rows of kF8Stride bytes: < 2^16)
    uint32_t offs[TPW];
    f32x16 acc[TPW];
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
        int ti, tj;
        tile_pair(pair0 + q < npairs ? pair0 + q : 0, nt, ti, tj);
        offs[q] = (uint32_t)((ti * kMT + rsub) * kF8Stride + kofs) |
                  ((uint32_t)((tj * kMT + rsub) * kF8Stride + kofs) << 16);
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[q][i] = 0.0f;
    }
    // the chunk is one contiguous block of rows x 64 bytes (padding rows are zero), read
    // as 16-byte pieces e = tid + 256 m into registers one chunk ahead
    static_assert(NWV * TPW == kPairsPerGroup, "a group holds kPairsPerGroup tile pairs");
    constexpr int kPieces = (kF8Rows * 4 + 64 * NWV - 1) / (64 * NWV);
    const int npieces = rows * 4;
    u32x4v reg[kPieces];
    double creg = 0.0;
    auto load_chunk = [&](int64_t kc) {
        const u32x4v *blk = reinterpret_cast<const u32x4v *>(u + (kc / kF8KC) * (int64_t)rows * kF8KC);
#pragma unroll
        for (int m = 0; m < kPieces; ++m) {
            const int e = threadIdx.x + 64 * NWV * m;
            u32x4v v = {0u, 0u, 0u, 0u};
            if (e < npieces) v = blk[e];
            reg[m] = v;
        }
        if (threadIdx.x < kF8KC) creg = c[kc + threadIdx.x];
    };
    if (k0 < k1) load_chunk(k0);
    for (int64_t kc = k0; kc < k1; kc += kF8KC) {
        if (threadIdx.x < kF8KC) cw[threadIdx.x] = (float)(sqrt(creg) * invS);
        __syncthreads();
        // decode, weight, re-encode into LDS; every piece of this thread covers the same
        // 16 rows of the chunk (piece = tid mod 4), so it needs 16 weights
        const int piece = threadIdx.x & 3;
        const float *wk = cw + 16 * piece;
#pragma unroll
        for (int m = 0; m < kPieces; ++m) {
            const int e = threadIdx.x + 64 * NWV * m;
            if (e < npieces) {
                const u32x4v raw = reg[m];
                u32x4v v;
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const int word = (int)raw[d];
                    int o = __builtin_amdgcn_cvt_pk_fp8_f32(__builtin_amdgcn_cvt_f32_fp8(word, 0) * wk[4 * d],
                                                            __builtin_amdgcn_cvt_f32_fp8(word, 1) * wk[4 * d + 1], 0,
                                                            false);
                    o = __builtin_amdgcn_cvt_pk_fp8_f32(__builtin_amdgcn_cvt_f32_fp8(word, 2) * wk[4 * d + 2],
                                                        __builtin_amdgcn_cvt_f32_fp8(word, 3) * wk[4 * d + 3], o, true);
                    v[d] = (unsigned)o;
                }
                *reinterpret_cast<u32x4v *>(sh8 + (e >> 2) * kF8Stride + 16 * piece) = v;
            }
        }
        __syncthreads();
        if (kc + kF8KC < k1) load_chunk(kc + kF8KC);   // in flight during the products below
        // a wave's pairs run along rows of the upper triangle: the A fragment (row tile ti) is
        // read from LDS only when ti changes
        i32x8v av;
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            if (q < nq) {
                if (q == 0 || (offs[q] & 0xffffu) != (offs[q - 1] & 0xffffu)) {
                    const uint8_t *pa = sh8 + (offs[q] & 0xffffu);
                    const u32x4v a0 = *reinterpret_cast<const u32x4v *>(pa);
                    const u32x4v a1 = *reinterpret_cast<const u32x4v *>(pa + 16);
                    av = i32x8v{(int)a0[0], (int)a0[1], (int)a0[2], (int)a0[3],
                                (int)a1[0], (int)a1[1], (int)a1[2], (int)a1[3]};
                }
                const uint8_t *pb = sh8 + (offs[q] >> 16);
                const u32x4v b0 = *reinterpret_cast<const u32x4v *>(pb), b1 = *reinterpret_cast<const u32x4v *>(pb + 16);
                const i32x8v bv = {(int)b0[0], (int)b0[1], (int)b0[2], (int)b0[3],
                                   (int)b1[0], (int)b1[1], (int)b1[2], (int)b1[3]};
                acc[q] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, acc[q], 0, 0, 0, 127, 0, 127);
            }
        }
        __syncthreads();   // the next chunk rewrites the LDS tiles
    }
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
        if (q < nq) {
            float *out = part + ((int64_t)s * npairs + pair0 + q) * (kMT * kMT);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int m = 8 * (i / 4) + 4 * (lane / 32) + (i % 4), n = lane % 32;
                out[m * kMT + n] = acc[q][i];
            }
        }
    }
}

// More than 10 row tiles in FP8: blocks of 8 x 8 tile pairs as in syrk_bf16_wide_kernel.  Per
// 128-row chunk (two of the copy's 64-row blocks) the rows of block I, and off the diagonal
// those of block J, are decoded, weighted and re-encoded into LDS -- both operands are the same
// matrix, so a diagonal block stages 256 rows only.  What bounds it is that conversion
// (8 vector instructions per 4 bytes, 2560 cycles per chunk and SIMD against 2050 of products):
// an element is converted once per block that it takes part in, 2 times at p = 500, where
// groups of 32 tile pairs that staged all rows converted it 5 times (N = 2.5e6: 1.22 -> 0.71 ms).
constexpr int kF8WideKC = 128, kF8WideStride = kF8WideKC + 16;

__global__ __launch_bounds__(64 * kWideWaves, 2) void syrk_fp8_wide_kernel(const uint8_t *u, int p, const double *c,
                                                                          const double *wsc, int64_t K,
                                                                          int64_t kchunk, float *part)
{
    extern __shared__ uint8_t sh8[];   // two buffers of [I rows, J rows][kF8WideStride]
    __shared__ float cw[2][kF8WideKC];
    constexpr int kHalf = kWideRows * kF8WideStride;
    const int nt = (p + kMT - 1) / kMT;
    const int rows = nt * kMT;
    const int nb = (nt + kWideTiles - 1) / kWideTiles;
    const int npairs = nt * (nt + 1) / 2;
    int I, J, s, grp;
    split_group(s, grp);
    tile_pair(grp, nb, I, J);
    const bool diag = I == J;
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t / 64);
    const int64_t k0 = (int64_t)s * kchunk;
    const int64_t k1 = k0 + kchunk < K ? k0 + kchunk : K;
    const double invS = 1.0 / wsc[0];
    const int piece = t % 8, row = t / 8;   // this thread's rows: row + 64 m; K values 16 piece ..
    u32x4v ra[kWidePer], rb[kWidePer];
    auto load = [&](int64_t kc) {
        const uint8_t *blk = u + (kc / kF8KC + piece / 4) * (int64_t)rows * kF8KC + 16 * (piece % 4);
        const bool in = kc + 16 * piece < k1;   // K is a multiple of 64
#pragma unroll
        for (int m = 0; m < kWidePer; ++m) {
            const int i = I * kWideRows + row + 64 * m, j = J * kWideRows + row + 64 * m;
            u32x4v va = {0u, 0u, 0u, 0u}, vb = {0u, 0u, 0u, 0u};
            if (in && i < rows) va = *reinterpret_cast<const u32x4v *>(blk + (int64_t)i * kF8KC);
            if (in && !diag && j < rows) vb = *reinterpret_cast<const u32x4v *>(blk + (int64_t)j * kF8KC);
            ra[m] = va;
            rb[m] = vb;
        }
    };
    auto weight = [&](int64_t k) { return k < k1 ? (float)(sqrt(c[k]) * invS) : 0.0f; };
    auto stage = [&](int buf, const float *cwk) {
        uint8_t *pa = sh8 + buf * 2 * kHalf + row * kF8WideStride + 16 * piece, *pb = pa + kHalf;
        float wk[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) wk[i] = cwk[16 * piece + i];
        auto convert = [&](const u32x4v &raw) {
            u32x4v v;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)raw[d], false);
                const auto hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)raw[d], true);
                int o = __builtin_amdgcn_cvt_pk_fp8_f32(lo[0] * wk[4 * d], lo[1] * wk[4 * d + 1], 0, false);
                o = __builtin_amdgcn_cvt_pk_fp8_f32(hi[0] * wk[4 * d + 2], hi[1] * wk[4 * d + 3], o, true);
                v[d] = (unsigned)o;
            }
            return v;
        };
#pragma unroll
        for (int m = 0; m < kWidePer; ++m) {
            *reinterpret_cast<u32x4v *>(pa + 64 * m * kF8WideStride) = convert(ra[m]);
            if (!diag) *reinterpret_cast<u32x4v *>(pb + 64 * m * kF8WideStride) = convert(rb[m]);
        }
    };
    f32x16 acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[q][i] = 0.0f;
    int wr, wc;
    const uint32_t want = wide_region(w, diag, wr, wc);
    const int frag = (lane & 31) * kF8WideStride + 32 * (lane >> 5);
    const uint8_t *fa = sh8 + 2 * wr * kMT * kF8WideStride + frag;
    const uint8_t *fb = sh8 + (diag ? 0 : kHalf) + 4 * wc * kMT * kF8WideStride + frag;
    auto products = [&](int buf) {
        const uint8_t *A = fa + buf * 2 * kHalf, *B = fb + buf * 2 * kHalf;
        auto get = [](const uint8_t *src) {
            const u32x4v x = *reinterpret_cast<const u32x4v *>(src), y = *reinterpret_cast<const u32x4v *>(src + 16);
            return i32x8v{(int)x[0], (int)x[1], (int)x[2], (int)x[3], (int)y[0], (int)y[1], (int)y[2], (int)y[3]};
        };
        if (want == 0u) return;
#pragma unroll
        for (int k = 0; k < kF8WideKC; k += kF8KC) {
            i32x8v a[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) a[i] = get(A + i * kMT * kF8WideStride + k);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const i32x8v b = get(B + j * kMT * kF8WideStride + k);
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (want & (1u << (4 * i + j)))
                        acc[4 * i + j] =
                            __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[i], b, acc[4 * i + j], 0, 0, 0, 127, 0, 127);
            }
        }
    };
    // the weights of chunk i + 2 replace those of chunk i once chunk i is staged
    double cnext = 0.0;
    if (t < kF8WideKC) {
        cw[0][t] = weight(k0 + t);
        cw[1][t] = weight(k0 + kF8WideKC + t);
        if (k0 + 2 * kF8WideKC + t < k1) cnext = c[k0 + 2 * kF8WideKC + t];
    }
    if (k0 < k1) load(k0);
    __syncthreads();
    if (k0 < k1) {
        stage(0, cw[0]);
        if (k0 + kF8WideKC < k1) load(k0 + kF8WideKC);
    }
    __syncthreads();
    int buf = 0;
    for (int64_t kc = k0; kc < k1; kc += kF8WideKC, buf ^= 1) {
        products(buf);
        if (kc + kF8WideKC < k1) {
            stage(buf ^ 1, cw[buf ^ 1]);   // last read before the previous barrier
            if (kc + 2 * kF8WideKC < k1) load(kc + 2 * kF8WideKC);
            if (t < kF8WideKC) {
                cw[buf][t] = (float)(sqrt(cnext) * invS);
                cnext = kc + 3 * kF8WideKC + t < k1 ? c[kc + 3 * kF8WideKC + t] : 0.0;
            }
        }
        __syncthreads();
    }
    const int64_t base = (int64_t)s * npairs;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int ti = I * kWideTiles + 2 * wr + q / 4, tj = J * kWideTiles + 4 * wc + q % 4;
        if ((want & (1u << q)) && ti < nt && tj < nt) store_tile(part, base + pair_index(ti, tj, nt), acc[q], lane);
    }
}

// C (+)= sign * scale_i * scale_j * sum over ranges of the partial tiles (FP64).
// Grid (npairs, 16): each workgroup takes 64 entries of one tile; its 16
// waves sum the splits q = w, w + 16, ... in order, then the 16 sums are
// added in wave order (a fixed order, so results do not vary run to run).
__global__ __launch_bounds__(64 * kRedWaves) void syrk_bf16_reduce_kernel(const float *part, int p, int S,
                                                                          const float *scale, double sign,
                                                                          int accumulate, double *C, const double *wsc)
{
    __shared__ double red[kRedWaves][64];
    const int nt = (p + kMT - 1) / kMT;
    const int npairs = nt * (nt + 1) / 2;
    const int pair = blockIdx.x;
    int ti, tj;
    tile_pair(pair, nt, ti, tj);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int e = blockIdx.y * 64 + lane;
    double s = 0.0;
    for (int q = w; q < S; q += kRedWaves) s += (double)part[((int64_t)q * npairs + pair) * (kMT * kMT) + e];
    red[w][lane] = s;
    __syncthreads();
    if (w != 0) return;
    s = red[0][lane];
    for (int v = 1; v < kRedWaves; ++v) s += red[v][lane];
    const int a = e / kMT, bb = e % kMT;
    const int i = ti * kMT + a, j = tj * kMT + bb;
    if (i >= p || j >= p) return;
    if (ti == tj && j < i) return;
    s *= sign * (double)scale[i] * (double)scale[j];
    if (wsc) s *= wsc[0] * wsc[0];
    if (accumulate) {
        C[(int64_t)i * p + j] += s;
        if (i != j) C[(int64_t)j * p + i] += s;
    } else {
        C[(int64_t)i * p + j] = s;
        if (i != j) C[(int64_t)j * p + i] = s;
    }
}

// xscale_j = the power of two s with max|x_j| / s <= xmax (1 for a zero column);
// zscale_j = the power of two >= max|x_j| (the BF16 scale of xbar_j).
__global__ __launch_bounds__(256) void colscale_kernel(const double *x, int64_t ld, float xmax, float *xscale,
                                                       float *zscale)
{
    __shared__ double red[4];
    const int j = blockIdx.x;
    double m = 0.0;
    for (int64_t r = threadIdx.x; r < ld; r += 256) m = fmax(m, fabs(x[(int64_t)j * ld + r]));
    for (int off = 32; off >= 1; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
        xscale[j] = m > 0.0 ? (float)exp2(ceil(log2(m / (double)xmax))) : 1.0f;
        zscale[j] = m > 0.0 ? (float)exp2(ceil(log2(m))) : 1.0f;
    }
}

__global__ __launch_bounds__(256) void to_bf16_kernel(const double *x, int64_t ld, const float *xscale,
                                                      uint16_t *xlp)
{
    const int j = blockIdx.y;
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r < ld) {
        const __hip_bfloat16 v = __float2bfloat16((float)(x[(int64_t)j * ld + r] / (double)xscale[j]));
        xlp[(int64_t)j * ld + r] = __builtin_bit_cast(uint16_t, v);
    }
}

}  // namespace

size_t syrk_bf16_partial_bytes(int p, int splits)
{
    return sizeof(float) * (size_t)splits * (size_t)npairs32(p) * kMT * kMT;
}

size_t syrk_partial_bytes(int p, int splits)
{
    const int nt = (p + kTile - 1) / kTile;
    return sizeof(double) * (size_t)splits * (size_t)(nt * (nt + 1) / 2) * kTile * kTile;
}

int syrk_f64(const double *u, int64_t ldu, int p, const double *c, int64_t K, int splits, double *part,
             double sign, int accumulate, double *C, hipStream_t stream)
{
    const int nt = (p + kTile - 1) / kTile;
    const int npairs = nt * (nt + 1) / 2;
    int64_t kchunk = (K + splits - 1) / splits;
    if (p <= 512 && ldu < (1 << 25)) {
        // matrix cores, every row of u staged once per K chunk: 2 * splits K ranges at p <= 256
        // (one group of blocks), splits ranges of 4 groups beyond; fewer ranges when K is short
        // (at least 4 chunks each), the reduction reading every range's tiles
        const int nb = (p + 15) / 16, ngroups = (nb * (nb + 1) / 2 + kF64Group - 1) / kF64Group;
        int s2 = p <= 256 ? 2 * splits : splits;
        const int64_t most = (K + 4 * kF64KC - 1) / (4 * kF64KC);
        if (most < s2) s2 = most > 1 ? (int)most : 1;
        if (ngroups > 1 && s2 >= 8) s2 = s2 / 8 * 8;   // whole groups of 8 ranges: one XCD runs all groups of a range
        kchunk = (K + s2 - 1) / s2;
        kchunk = (kchunk + kF64KC - 1) / kF64KC * kF64KC;
#define COXMI_SYRKF64(MB) \
    syrk_f64_mfma_kernel<MB><<<dim3(s2, ngroups), 64 * kF64Waves, 0, stream>>>(u, ldu, p, c, K, kchunk, part)
        if (nb > 16) COXMI_SYRKF64(32);
        else if (nb > 12) COXMI_SYRKF64(16);
        else if (nb > 8) COXMI_SYRKF64(12);
        else if (nb > 4) COXMI_SYRKF64(8);
        else if (nb > 2) COXMI_SYRKF64(4);
        else if (nb > 1) COXMI_SYRKF64(2);
        else COXMI_SYRKF64(1);
#undef COXMI_SYRKF64
        syrk_reduce_kernel<<<dim3(npairs, kTile * kTile / 64), 64 * kRedWaves, 0, stream>>>(part, p, s2, sign,
                                                                                           accumulate, C);
        return hipGetLastError() == hipSuccess ? 0 : -3;
    }
    kchunk = (kchunk + kKc - 1) / kKc * kKc;
    syrk_f64_kernel<<<dim3(npairs, splits), kSyrkThreads, 0, stream>>>(u, ldu, p, c, K, kchunk, part);
    syrk_reduce_kernel<<<dim3(npairs, kTile * kTile / 64), 64 * kRedWaves, 0, stream>>>(part, p, splits, sign,
                                                                                       accumulate, C);
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

int make_bf16_copy(const double *x, int64_t ld, int p, void *xlp, float *xscale, float *zscale, hipStream_t stream)
{
    colscale_kernel<<<p, 256, 0, stream>>>(x, ld, 1.0f, xscale, zscale);
    to_bf16_kernel<<<dim3((unsigned)((ld + 255) / 256), p), 256, 0, stream>>>(x, ld, xscale,
                                                                             static_cast<uint16_t *>(xlp));
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

namespace {

template <bool WEIGHT, bool BLK>
int launch_syrk_bf16(const uint16_t *u, int64_t ldu, int p, const double *c, int64_t K64, int *splits, float *part,
                     hipStream_t stream)
{
    const int nt = (p + kMT - 1) / kMT;
    if (nt <= 8) {
        // two workgroups per compute unit, 64-row chunks (at most 72 KB of LDS each, 8 tiles with the weighted copy)
        const int ngroups = (npairs32(p) + kPairsPerGroup - 1) / kPairsPerGroup;
        *splits *= 2;
        int64_t kchunk = (K64 + *splits - 1) / *splits;
        kchunk = (kchunk + 63) / 64 * 64;
        constexpr size_t per_tile = sizeof(uint16_t) * kMT * (64 + 8) * (WEIGHT ? 2 : 1);
        auto *fn = &syrk_bf16_lds_kernel<WEIGHT, BLK, 64, 8, 4, 8, 4>;
        static LdsLimit limit;
        if (limit.raise(reinterpret_cast<const void *>(fn), 8 * per_tile) != hipSuccess) return -3;
        fn<<<dim3(*splits, ngroups), 64 * 8, nt * per_tile, stream>>>(u, ldu, p, c, K64, kchunk, part);
    } else {
        const int nb = (nt + kWideTiles - 1) / kWideTiles;
        const int nblocks = nb * (nb + 1) / 2;
        if (*splits * (int64_t)nblocks > 16384) *splits = 16384 / nblocks > 1 ? 16384 / nblocks : 1;
        int64_t kchunk = (K64 + *splits - 1) / *splits;
        kchunk = (kchunk + kWideKC - 1) / kWideKC * kWideKC;
        constexpr size_t lds = sizeof(uint16_t) * (size_t)4 * kWideRows * kWideStride;
        auto *fn = &syrk_bf16_wide_kernel<WEIGHT, BLK>;
        static LdsLimit limit;
        if (limit.raise(reinterpret_cast<const void *>(fn), lds) != hipSuccess) return -3;
        fn<<<dim3(*splits, nblocks), 64 * kWideWaves, lds, stream>>>(u, ldu, p, c, K64, kchunk, part);
    }
    return 0;
}

}  // namespace

int syrk_bf16(const uint16_t *u, int64_t ldu, int p, bool blocked, const float *scale, const double *c, int64_t K,
              int splits, double *part, double sign, int accumulate, double *C, hipStream_t stream)
{
    const int64_t K64 = (K + 63) / 64 * 64;   // entries K..K64-1 are zero (padding)
    if (ldu % 64 != 0 || K64 > ldu || (blocked && c)) return -1;
    float *fpart = reinterpret_cast<float *>(part);
    int rc;
    if (c) rc = launch_syrk_bf16<true, false>(u, ldu, p, c, K64, &splits, fpart, stream);
    else if (blocked) rc = launch_syrk_bf16<false, true>(u, ldu, p, c, K64, &splits, fpart, stream);
    else rc = launch_syrk_bf16<false, false>(u, ldu, p, c, K64, &splits, fpart, stream);
    if (rc != 0) return rc;
    // sums the slices that the launch wrote
    syrk_bf16_reduce_kernel<<<dim3(npairs32(p), 16), 64 * kRedWaves, 0, stream>>>(fpart, p, splits, scale, sign,
                                                                                 accumulate, C, nullptr);
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

namespace {

int compute_units()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    return cus;
}

}  // namespace

size_t fp8_copy_bytes(int64_t ld, int p)
{
    return (size_t)ld * (size_t)((p + kMT - 1) / kMT * kMT);
}

int make_fp8_copy(const double *x, int64_t ld, int p, uint8_t *x8, float *xscale, float *zscale, hipStream_t stream)
{
    if (ld % kF8KC != 0) return -1;
    const int prow = (p + kMT - 1) / kMT * kMT;
    colscale_kernel<<<p, 256, 0, stream>>>(x, ld, kFp8Max, xscale, zscale);
    to_fp8_kernel<<<dim3((unsigned)((ld / 4 + 255) / 256), prow), 256, 0, stream>>>(x, ld, p, prow, xscale, x8);
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

int syrk_fp8(const uint8_t *u, int64_t ldu, int p, const float *scale, const double *c, int64_t K, int splits,
             double *part, double *blockmax, double *wsc, double sign, int accumulate, double *C, hipStream_t stream)
{
    const int nt = (p + kMT - 1) / kMT;
    const int npairs = nt * (nt + 1) / 2;
    const int ngroups = (npairs + kPairsPerGroup - 1) / kPairsPerGroup;
    const int64_t K64 = (K + kF8KC - 1) / kF8KC * kF8KC;
    if (K64 > ldu || ldu % kF8KC != 0) return -1;
    bmax_kernel<<<256, 256, 0, stream>>>(c, K, blockmax);
    wscale_kernel<<<1, 256, 0, stream>>>(blockmax, 256, wsc);
    if (nt * kMT > kF8Rows) {
        const int nb = (nt + kWideTiles - 1) / kWideTiles;
        const int nblocks = nb * (nb + 1) / 2;
        int bsplits = splits;
        if (bsplits * (int64_t)nblocks > 16384) bsplits = 16384 / nblocks > 1 ? 16384 / nblocks : 1;
        // A range's partials are written and read whatever its length: at least 8 chunks to a range, but
        // a workgroup for every compute unit (N = 2e4, P = 800: 437 us with 256 ranges of one chunk
        // and the product of Z, 274 with 24 of seven; the one-pass kernel 333)
        const int per_cu = compute_units() / nblocks, by_length = (int)(K64 / (8 * kF8WideKC));
        const int most = by_length > per_cu ? by_length : per_cu;
        if (most < bsplits) bsplits = most >= 8 ? most / 8 * 8 : (most > 1 ? most : 1);
        int64_t kchunk = (K64 + bsplits - 1) / bsplits;
        kchunk = (kchunk + kF8WideKC - 1) / kF8WideKC * kF8WideKC;
        const size_t lds = (size_t)4 * kWideRows * kF8WideStride;
        static LdsLimit limit;
        if (limit.raise(reinterpret_cast<const void *>(&syrk_fp8_wide_kernel), lds) != hipSuccess) return -3;
        float *fpart = reinterpret_cast<float *>(part);
        syrk_fp8_wide_kernel<<<dim3(bsplits, nblocks), 64 * kWideWaves, lds, stream>>>(u, p, c, wsc, K64, kchunk, fpart);
        syrk_bf16_reduce_kernel<<<dim3(npairs, 16), 64 * kRedWaves, 0, stream>>>(fpart, p, bsplits, scale, sign, accumulate, C,
                                                                     wsc);
        return hipGetLastError() == hipSuccess ? 0 : -3;
    }
    // two workgroups per compute unit are resident: size the grid to whole rounds of them
    int fit = (4 * compute_units()) / ngroups;
    if (fit >= 8) fit = fit / 8 * 8;   // whole groups of 8 K ranges: one XCD runs all groups of a range
    if (fit >= 1 && fit < splits) splits = fit;
    int64_t kchunk = (K64 + splits - 1) / splits;
    kchunk = (kchunk + kF8KC - 1) / kF8KC * kF8KC;
    const size_t lds = (size_t)nt * kMT * kF8Stride;
    float *fpart = reinterpret_cast<float *>(part);
    syrk_fp8_lds_kernel<><<<dim3(splits, ngroups), 64 * kSyrkBfWaves, lds, stream>>>(u, p, c, wsc, K64, kchunk, fpart);
    syrk_bf16_reduce_kernel<<<dim3(npairs, 16), 64 * kRedWaves, 0, stream>>>(fpart, p, splits, scale, sign, accumulate, C, wsc);
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

// Proximal Newton's model solve: cyclic coordinate descent with soft thresholding (the l1
// rule of Sec. 2.4, applied to the quadratic model of the objective)
//   min_D  g'D + D'HD/2 + sum_j gamma_j |beta_j + D_j|
// in one workgroup.  With z_j = beta_j + D_j, a_j = H_jj and v_j = sum_{i != j} H_ji D_i, coordinate
// j moves to soft(u_j, gamma_j) / a_j where u_j = a_j beta_j - g_j - v_j; a move of another coordinate
// i by delta adds H_ij delta to v_j.  The parts that stay (a_j beta_j - g_j -+ gamma_j) are rounded
// once and v alone takes the moves: it is as small as D, so a move rounds at the size of the moves,
// not at that of a_j beta_j (with u itself carried along, an AR(1) fit of 300 columns ended 3e-14
// from the model's minimum, now 5e-16).  Coordinates not free, or with H_jj <= 0 or not finite,
// stay, and their rows of H, which may hold NaN or infinities, are not read.  Stops after the first
// sweep whose largest |change| is <= tol, or after max_sweeps sweeps.
//
// The chain is what bounds it: each coordinate needs the one before.  Coordinates go in blocks
// of 64: wave 0 holds a block's v in its lanes and takes its 64 decisions in turn from the
// 64 x 64 diagonal block in LDS (7 dependent FP64 operations and a lane broadcast each), while the
// other waves stage the next diagonal block; then all 16 waves apply the block's moves to the
// rest of v, a row of H per moved coordinate, 32 rows in flight.  One wave that
// fetched a row of H per coordinate (a memory round trip each) took 9.9 ms per solve in a
// p = 1000 fit; this takes 2.0 ms.
constexpr int kProxB = 64;         // coordinates of a block
constexpr int kProxThreads = 1024;
constexpr int kProxRows = 32;      // rows of H in flight per thread

__global__ __launch_bounds__(kProxThreads) void prox_cd_kernel(const double *H, int p, const double *g,
                                                               const double *beta, const double *gam,
                                                               const uint8_t *free_col, double tol, int max_sweeps,
                                                               double *D, int *sweeps_out)
{
    extern __shared__ double sm[];   // v[p], z[p], two diagonal blocks (row-major, zero diagonal)
    double *v = sm, *z = sm + p, *blk = sm + 2 * (size_t)p;
    __shared__ double s_delta[kProxB];
    __shared__ int s_row[kProxB], s_moved;
    __shared__ double s_change;
    __shared__ unsigned long long s_live[kMaxNewtonP / kProxB];   // a bit per coordinate: it may move
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t / 64);
    const int nblk = (p + kProxB - 1) / kProxB;
    for (int b = w; b < nblk; b += kProxThreads / 64) {
        const int j = b * kProxB + lane;
        const double a = j < p ? H[(size_t)j * p + j] : 0.0;
        const unsigned long long mask = __builtin_amdgcn_ballot_w64(j < p && free_col[j] && a > 0.0 && a < INFINITY);
        if (lane == 0) s_live[b] = mask;
    }
    __syncthreads();
    // (the decisions subtract row i times coordinate i's move, 0 for one that stays: 0 times NaN)
    auto stage = [&](int block, int first, int threads) {
        double *dst = blk + (block & 1) * (kProxB * kProxB);
        const int j0 = block * kProxB;
        for (int e = t - first; e < kProxB * kProxB; e += threads) {
            const int r = e / kProxB, c = e % kProxB;
            dst[e] = (r != c && ((s_live[block] >> r) & 1ull) && j0 + c < p) ? H[(size_t)(j0 + r) * p + j0 + c] : 0.0;
        }
    };
    for (int k = t; k < p; k += kProxThreads) {
        v[k] = 0.0;
        z[k] = beta[k];
    }
    stage(0, 0, kProxThreads);
    // wave 0's inputs of its lane's coordinate, one block ahead: a beta - g -+ gamma and 1 / a (0: it stays)
    double lo = 0.0, hi = 0.0, inv = 0.0;
    auto inputs = [&](int block, double &l, double &h, double &iv) {
        const int j = block * kProxB + lane;
        l = h = iv = 0.0;
        if ((s_live[block] >> lane) & 1ull) {
            const double a = H[(size_t)j * p + j], c = fma(a, beta[j], -g[j]), gm = gam[j];
            l = c - gm;
            h = c + gm;
            iv = 1.0 / a;
        }
    };
    if (w == 0) inputs(0, lo, hi, inv);
    int sweep = 0;
    while (sweep < max_sweeps) {
        ++sweep;
        double change = 0.0;   // wave 0's lanes
        for (int b = 0; b < nblk; ++b) {
            const int nextb = b + 1 < nblk ? b + 1 : 0;
            const int j0 = b * kProxB, nb = p - j0 < kProxB ? p - j0 : kProxB;
            // one block stays where it is; with an odd number the first one's buffer is the last one's too
            const bool restage = nblk > 1, clash = restage && nextb == 0 && (b & 1) == 0;
            __syncthreads();   // v holds every earlier move, the diagonal block is staged
            if (w == 0) {
                double lon, hin, invn;
                inputs(nextb, lon, hin, invn);   // in flight during the decisions
                const bool live = lane < nb && inv != 0.0;
                double vl = lane < nb ? v[j0 + lane] : 0.0, zl = lane < nb ? z[j0 + lane] : 0.0;
                double moved = 0.0;
                const double *row = blk + (b & 1) * (kProxB * kProxB) + lane;
                double hc[8], hn[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) hc[q] = row[q * kProxB];
                for (int i0 = 0; i0 < nb; i0 += 8) {
                    const int in = i0 + 8 < kProxB ? i0 + 8 : 0;
#pragma unroll
                    for (int q = 0; q < 8; ++q) hn[q] = row[(in + q) * kProxB];
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        // every lane's move as of now; lane i0 + q takes its own
                        const double soft = vl < lo ? lo - vl : (vl > hi ? hi - vl : 0.0);
                        const double znew = live ? soft * inv : zl;
                        const double delta = lane_value(znew - zl, i0 + q);
                        if (lane == i0 + q) {
                            moved = znew - zl;
                            zl = znew;
                        }
                        vl = fma(hc[q], delta, vl);
                    }
#pragma unroll
                    for (int q = 0; q < 8; ++q) hc[q] = hn[q];
                }
                if (lane < nb) {
                    v[j0 + lane] = vl;
                    z[j0 + lane] = zl;
                }
                change = fmax(change, fabs(moved));
                // the moved coordinates, in order
                const unsigned long long mask = __builtin_amdgcn_ballot_w64(moved != 0.0);
                if (moved != 0.0) {
                    const int at = __popcll(mask & ((1ull << lane) - 1ull));
                    s_delta[at] = moved;
                    s_row[at] = j0 + lane;
                }
                if (lane == 0) s_moved = __popcll(mask);
                lo = lon;
                hi = hin;
                inv = invn;
            } else if (restage && !clash) {
                stage(nextb, 64, kProxThreads - 64);
            }
            __syncthreads();
            const int m = s_moved;
            for (int k = t; k < p; k += kProxThreads) {
                if (k >= j0 && k < j0 + nb) continue;
                double acc = v[k];
                for (int q0 = 0; q0 < m; q0 += kProxRows) {
                    double h[kProxRows];
#pragma unroll
                    for (int q = 0; q < kProxRows; ++q) {
                        const int r = s_row[q0 + q < m ? q0 + q : q0];
                        h[q] = H[(size_t)r * p + k];
                    }
#pragma unroll
                    for (int q = 0; q < kProxRows; ++q)
                        if (q0 + q < m) acc = fma(h[q], s_delta[q0 + q], acc);
                }
                v[k] = acc;
            }
            if (clash) stage(nextb, 0, kProxThreads);   // nobody reads the buffer before the next barrier
        }
        if (w == 0) {
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) change = fmax(change, __shfl_xor(change, o, 64));
            if (lane == 0) s_change = change;
        }
        __syncthreads();
        const double most = s_change;
        if (most <= tol) break;
    }
    __syncthreads();
    for (int k = t; k < p; k += kProxThreads) D[k] = z[k] - beta[k];
    if (t == 0) *sweeps_out = sweep;
}

int prox_model_solve(const double *H, int p, const double *g, const double *beta, const double *gam,
                     const uint8_t *free_col, double tol, int max_sweeps, double *D, int *sweeps, hipStream_t stream)
{
    if (p < 1 || p > 4096) return -1;
    const size_t lds = sizeof(double) * (2 * (size_t)p + 2 * kProxB * kProxB);
    static LdsLimit limit;
    if (limit.raise(reinterpret_cast<const void *>(&prox_cd_kernel),
                    sizeof(double) * (2 * kMaxNewtonP + 2 * kProxB * kProxB)) != hipSuccess)
        return -3;
    prox_cd_kernel<<<1, kProxThreads, lds, stream>>>(H, p, g, beta, gam, free_col, tol, max_sweeps, D, sweeps);
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

int chol_solve(double *A, int p, const double *g, const uint8_t *free_col, int factored, double *dx, int *status,
               hipStream_t stream)
{
    auto tail_lds = [](int n) { return sizeof(double) * ((size_t)n * (n + 1) / 2 + kTriPad + n); };
    static LdsLimit tail_limit, solve_limit;
    if (tail_limit.raise(reinterpret_cast<const void *>(&chol_tail_kernel), tail_lds(kCholTail)) != hipSuccess ||
        solve_limit.raise(reinterpret_cast<const void *>(&chol_solve_kernel), sizeof(double) * 8192) != hipSuccess)
        return -3;
    auto tail = [&](int r0) {
        const int n = p - r0;
        // four waves have enough tiles up to 64 columns, and their barriers are shorter
        chol_tail_kernel<<<1, n <= kBlk ? 256 : kTailThreads, tail_lds(n), stream>>>(A, p, r0, g, free_col, factored, dx, status);
    };
    if (p <= kCholTail) {
        tail(0);
    } else {
        if (!factored) {
            auto tiles = [&](int r0) {
                const int nt = (p - r0 + kBlk - 1) / kBlk;
                return (unsigned)(nt * (nt + 1) / 2);
            };
            chol_tile_kernel<<<tiles(0), 256, 0, stream>>>(A, p, -1, 0, free_col, 1);
            int r0 = 0;
            while (p - r0 > kCholTail) {
                chol_rows_kernel<<<(unsigned)((p - r0 - 1) / kBlk), 256, 0, stream>>>(A, p, r0);
                r0 += kBlk;
                chol_tile_kernel<<<tiles(r0), 256, 0, stream>>>(A, p, r0 - kBlk, r0, free_col, p - r0 > kCholTail);
            }
            tail(r0);
        }
        chol_solve_kernel<<<1, kSolveThreads, sizeof(double) * (size_t)p, stream>>>(A, p, g, free_col, dx, status);
    }
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

}  // namespace coxmi
