// newton.hip -- full evaluation of the stratified Cox objective, gradient and
// information matrix on gfx950, and the FP64 Cholesky solve of a Newton step.
//
// Exchanging the order of the sums in Eqs. strat_g / strat_h (every event
// group g adds d_g x_r w_r / S0_g for each row r of its risk set) gives, with
// Lambda_r = sum over the event groups g of r's stratum with Y_g <= Y_r of
// d_g / S0_g (a reverse segmented scan of d_g / S0_g):
//   gradient     = X'(w o Lambda - delta)
//   Hessian      = X' diag(w o Lambda) X - sum_g d_g xbar_g xbar_g',  xbar_g = S1_g / S0_g
//   diagonal     = sum_r x_rj^2 w_r Lambda_r - sum_g d_g xbar_gj^2
//   objective    = -delta'eta + sum_g d_g (log S0_g + c)
// where S0_g, S1_g are the forward segmented scans of w and w x at the end of
// group g, w = exp(eta - c).  One pass over X forms eta, one more forms the
// X' products, and one per-column scan forms xbar; the information matrix is
// two symmetric rank-K products (contraction.hip).
//
// Efron's tie correction (Efron 1977; the paper's risk sets are Breslow's): the l-th of the
// d events of group g sees A_l = S0_g - (l/d) E0_g, E the sums over the group's own events.
// With h_g = sum_l 1/A_l and k_g = sum_l (l/d)/A_l the same exchange of sums gives
//   gradient     = X'(w o c - delta),  c_r = sum_{g: r in R_g} h_g - delta_r k_{g(r)}
//   Hessian      = X' diag(w o c) X - sum_g [S1 E1] M_g [S1 E1]',  M_g = sum_l (1, -a_l)(1, -a_l)' / A_l^2
//   objective    = -delta'eta + sum_g sum_l (log A_l + c)
// and M_g = L L' (2 x 2 Cholesky) turns each group's term into two rows of Z: l11 S1 + l21 E1
// and l22 E1.  For d = 1, a_0 = 0 and these are the plain terms (h = 1/S0, one row S1/S0), so
// E1 is needed only for the groups with two or more events, whose event rows are listed.
//
// All kernels here are ordinary launches (no cross-workgroup waits).
#include <hip/hip_bf16.h>
#include <math.h>

#include <cmath>

#include <type_traits>

#include "internal.h"
#include "newton.h"
#include "affscan.hpp"
#include "segscan.hpp"

namespace coxmi {

namespace {

constexpr int kRowBlock = 256;   // threads of the elementwise and reduction kernels

__device__ __forceinline__ double block_sum(double v, double *red)
{
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    if (lane == 0) red[w] = v;
    __syncthreads();
    double s = 0.0;
    for (int k = 0; k < (int)(blockDim.x / kWave); ++k) s += red[k];
    __syncthreads();
    return s;
}

__device__ __forceinline__ double block_max(double v, double *red)
{
    for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off, kWave));
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    if (lane == 0) red[w] = v;
    __syncthreads();
    double s = -INFINITY;
    for (int k = 0; k < (int)(blockDim.x / kWave); ++k) s = fmax(s, red[k]);
    __syncthreads();
    return s;
}

// eta = X beta over all ld rows.
__global__ __launch_bounds__(kRowBlock) void eta_kernel(const double *x, int64_t ld, int p, const double *beta,
                                                        double *eta)
{
    const int64_t r = (int64_t)blockIdx.x * kRowBlock + threadIdx.x;
    if (r < ld) {
        double e = 0.0;
        for (int j = 0; j < p; ++j) {
            const double bj = beta[j];
            if (bj != 0.0) e = fma(x[(int64_t)j * ld + r], bj, e);
        }
        eta[r] = e;
    }
}

// With m the running maximum of eta within the stratum: alpha_r =
// exp(m_{r-1} - m_r) (1 at a head) and u_r = exp(eta_r - m_r), both in (0, 1].
__global__ __launch_bounds__(kRowBlock) void prep_kernel(const double *eta, const double *m, const uint32_t *meta,
                                                         int64_t ld, double *alpha, double *u)
{
    const int64_t r = (int64_t)blockIdx.x * kRowBlock + threadIdx.x;
    if (r < ld) {
        const double mr = m[r];
        alpha[r] = (meta[r] & kHeadBit) ? 1.0 : exp(m[r - 1] - mr);
        u[r] = exp(eta[r] - mr);
    }
}

// At event-group ends, with S0' = S0 exp(-m) in [1, n]: h' = d / S0', its
// objective part d (log S0' + m), and zq = h' / sqrt(d) (so that
// sqrt(d) xbar_j = S1'_j zq and d xbar_j^2 = (S1'_j zq)^2: no division per
// column); -eta at event rows.  A non-finite S0' (non-finite X beta) is flagged.
__global__ __launch_bounds__(kRowBlock) void hazard_kernel(const double *s0, const double *eta, const double *m,
                                                           const uint32_t *meta, int64_t ld, double *h, double *zq,
                                                           double *blockobj, unsigned *flags)
{
    __shared__ double red[kRowBlock / kWave];
    const int64_t r = (int64_t)blockIdx.x * kRowBlock + threadIdx.x;
    double obj = 0.0;
    if (r < ld) {
        const uint32_t mw = meta[r];
        const uint32_t d = mw & kCountMask;
        double hv = 0.0, qv = 0.0;
        if (d != 0u) {
            const double s = s0[r];
            if (!(s >= 0.5) || !(s <= 1e300)) atomicOr(flags, 1u);
            hv = (double)d / s;
            qv = hv / sqrt((double)d);
            obj += (double)d * (log(s) + m[r]);
        }
        if (mw & kEventBit) obj -= eta[r];
        h[r] = hv;
        zq[r] = qv;
    }
    obj = block_sum(obj, red);
    if (threadIdx.x == 0) blockobj[blockIdx.x] = obj;
}

// b = w Lambda = u R, with R the reverse recurrence of h' (relative to exp(m_r))
__global__ __launch_bounds__(kRowBlock) void rowweight_kernel(const double *u, const double *R, int64_t ld, double *b)
{
    const int64_t r = (int64_t)blockIdx.x * kRowBlock + threadIdx.x;
    if (r < ld) b[r] = u[r] * R[r];
}

// Efron at event-group ends, everything relative to exp(m_r) as above: A'_l = S0' - (l/d) E0',
// h' = sum_l 1/A'_l, k' = sum_l (l/d)/A'_l, objective sum_l (log A'_l + m), and the factor of
// M' = sum_l (1, -a_l)(1, -a_l)' / A'_l^2 (l11 in zq, l21, l22); -eta at event rows.
__global__ __launch_bounds__(kRowBlock) void hazard_efron_kernel(const double *s0, const double *e0, const double *eta,
                                                                 const double *m, const uint32_t *meta, int64_t ld,
                                                                 double *h, double *kq, double *zq, double *zq2,
                                                                 double *zq3, double *blockobj, unsigned *flags)
{
    __shared__ double red[kRowBlock / kWave];
    const int64_t r = (int64_t)blockIdx.x * kRowBlock + threadIdx.x;
    double obj = 0.0;
    if (r < ld) {
        const uint32_t mw = meta[r];
        const uint32_t d = mw & kCountMask;
        double hv = 0.0, kv = 0.0, l11 = 0.0, l21 = 0.0, l22 = 0.0;
        if (d != 0u) {
            const double s = s0[r], ev = e0[r], mr = m[r], dd = (double)d;
            if (!(s >= 0.5) || !(s <= 1e300)) atomicOr(flags, 1u);
            double m11 = 0.0, m21 = 0.0, m22 = 0.0;
            for (uint32_t l = 0; l < d; ++l) {
                const double a = (double)l / dd;
                const double A = s - a * ev;
                const double iA = 1.0 / A, iA2 = iA * iA;
                hv += iA;
                kv += a * iA;
                m11 += iA2;
                m21 -= a * iA2;
                m22 += a * a * iA2;
                obj += log(A) + mr;
            }
            l11 = sqrt(m11);
            l21 = m21 / l11;
            l22 = sqrt(fmax(m22 - l21 * l21, 0.0));
        }
        if (mw & kEventBit) obj -= eta[r];
        h[r] = hv;
        kq[r] = kv;
        zq[r] = l11;
        zq2[r] = l21;
        zq3[r] = l22;
    }
    obj = block_sum(obj, red);
    if (threadIdx.x == 0) blockobj[blockIdx.x] = obj;
}

// b = w c = u R - delta exp(eta - m_e) k'_e, e the end row of the row's tie group
__global__ __launch_bounds__(kRowBlock) void rowweight_efron_kernel(const double *u, const double *R, const double *eta,
                                                                    const double *m, const double *kq,
                                                                    const int32_t *gend, int64_t ld, double *b)
{
    const int64_t r = (int64_t)blockIdx.x * kRowBlock + threadIdx.x;
    if (r < ld) {
        double v = u[r] * R[r];
        const int32_t e = gend[r];
        if (e >= 0) v -= exp(eta[r] - m[e]) * kq[e];
        b[r] = v;
    }
}

// me_w[q] = exp(eta - m_end) of the listed event rows of the multi-event groups
__global__ __launch_bounds__(kRowBlock) void efron_w_kernel(const double *eta, const double *m, const int32_t *me_ptr,
                                                            const int32_t *me_row, const int32_t *me_end,
                                                            int64_t n_multi, double *me_w)
{
    const int64_t k = (int64_t)blockIdx.x * kRowBlock + threadIdx.x;
    if (k < n_multi) {
        const double me = m[me_end[k]];
        for (int32_t q = me_ptr[k]; q < me_ptr[k + 1]; ++q) me_w[q] = exp(eta[me_row[q]] - me);
    }
}

template <typename ZT>
__device__ __forceinline__ void store_z(ZT *p, double v, float inv_scale)
{
    if constexpr (std::is_same<ZT, double>::value) *p = v;
    else if constexpr (std::is_same<ZT, float>::value) *p = (float)v * inv_scale;
    else *p = __float2bfloat16((float)v * inv_scale);
}

// ------------------------------------------------------------------ column pass
//
// Rows are cut into tiles of `tile` rows (the persistent kernel's tiles, so in
// the stratum-aligned layout most tiles start with a stratum head).  One wave
// handles one (tile, column): the forward segmented scan of w x_j over the
// tile's rows (S1, carried in from the previous tiles when the tile's first
// row continues a stratum), xbar = S1/S0 at event-group ends with
// z = sqrt(d) xbar and sum d xbar^2, and the tile's parts of x'(w Lambda - delta)
// and (x o x)'(w Lambda).  The carries come from a masked sum per (tile,
// column) -- the rows after the tile's last head -- chained per column.

constexpr int kColWaves = 4, kColIpt = 4, kColChunk = kWave * kColIpt;

__device__ __forceinline__ void load4(const double *p, double *v)
{
    const double2 lo = *reinterpret_cast<const double2 *>(p);
    const double2 hi = *reinterpret_cast<const double2 *>(p + 2);
    v[0] = lo.x;
    v[1] = lo.y;
    v[2] = hi.x;
    v[3] = hi.y;
}

// The map S -> A S + B of the rows of tile t from its last head (or its first row) to its
// end for the recurrence S'_r = alpha_r S'_{r-1} + u_r x_rj, for the tiles listed in `tiles`.
// Unrolled, B = sum_r W_r x_rj with W_r = u_r times the alphas after r, which no column changes:
// colweight_kernel forms W and A, one workgroup per tile, and
// colagg_kernel is then a product of X with it, bound by reading X (200,000 x 100: 34 us at
// the rate of a copy).  A scan per column and tile took 79 us there, the two kernels 32.
constexpr int kWeightBlock = 256;

__global__ __launch_bounds__(kWeightBlock) void colweight_kernel(const double *alpha, const double *u, int64_t tile,
                                                                 const int32_t *tiles, const int32_t *lasthead,
                                                                 double *wsuf, double *taila)
{
    __shared__ double s_p[2][kWeightBlock];
    const int t = tiles[blockIdx.x], i = threadIdx.x;
    const int64_t r1 = (int64_t)(t + 1) * tile;
    const int64_t r0 = lasthead[t] >= 0 ? (int64_t)lasthead[t] : (int64_t)t * tile;
    const int64_t per = (r1 - r0 + kWeightBlock - 1) / kWeightBlock;
    const int64_t a = r0 + i * per < r1 ? r0 + i * per : r1, e = a + per < r1 ? a + per : r1;
    double prod = 1.0;
    for (int64_t r = a; r < e; ++r) prod *= alpha[r];
    s_p[0][i] = prod;
    int cur = 0;
    for (int o = 1; o < kWeightBlock; o *= 2, cur ^= 1) {
        __syncthreads();
        s_p[cur ^ 1][i] = i + o < kWeightBlock ? s_p[cur][i] * s_p[cur][i + o] : s_p[cur][i];
    }
    __syncthreads();
    double run = i + 1 < kWeightBlock ? s_p[cur][i + 1] : 1.0;   // the alphas after this thread's rows
    for (int64_t r = e - 1; r >= a; --r) {
        wsuf[r] = u[r] * run;
        run *= alpha[r];
    }
    if (i == 0) taila[t] = run;
}

// One wave per tile and 4 columns.
constexpr int kAggCols = 4;

__global__ __launch_bounds__(kWave * kColWaves) void colagg_kernel(const double *x, int64_t ld, int p, const double *wsuf,
                                                                   int64_t tile, const int32_t *tiles, int ntl,
                                                                   const int32_t *lasthead, double *aggb)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int groups = (p + kAggCols - 1) / kAggCols;
    const int item = __builtin_amdgcn_readfirstlane(blockIdx.x * kColWaves + threadIdx.x / kWave);
    if (item >= ntl * groups) return;
    const int t = tiles[item / groups], j0 = (item % groups) * kAggCols;
    const int64_t start = (int64_t)t * tile, r1 = start + tile;
    const int64_t r0 = lasthead[t] >= 0 ? (int64_t)lasthead[t] : start;
    constexpr int kRows = 2 * kWave;   // two rows per lane and load
    const double *xj[kAggCols];
    double acc[kAggCols];
#pragma unroll
    for (int c = 0; c < kAggCols; ++c) {
        xj[c] = x + (int64_t)(j0 + c < p ? j0 + c : p - 1) * ld;
        acc[c] = 0.0;
    }
#pragma unroll 4
    for (int64_t base = start + (r0 - start) / kRows * kRows; base < r1; base += kRows) {
        const int64_t r = base + 2 * lane;
        if (r + 1 < r1 && r >= r0) {
            const double2 w = *reinterpret_cast<const double2 *>(wsuf + r);
#pragma unroll
            for (int c = 0; c < kAggCols; ++c) {
                const double2 v = *reinterpret_cast<const double2 *>(xj[c] + r);
                acc[c] = fma(w.y, v.y, fma(w.x, v.x, acc[c]));
            }
        } else {   // the pair at the last head or at an odd end
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (r + k >= r0 && r + k < r1)
#pragma unroll
                    for (int c = 0; c < kAggCols; ++c) acc[c] = fma(wsuf[r + k], xj[c][r + k], acc[c]);
        }
    }
#pragma unroll
    for (int c = 0; c < kAggCols; ++c) {
#pragma unroll
        for (int o = kWave / 2; o >= 1; o >>= 1) acc[c] += __shfl_xor(acc[c], o, kWave);
        if (lane == 0 && j0 + c < p) aggb[(int64_t)t * p + j0 + c] = acc[c];
    }
}

// carry[t][j] = S'_j entering tile t (for tiles whose first row continues a stratum): one
// wave per column scans the tiles' maps, 64 at a time.  (A thread per column, tile after tile,
// waited for memory at every one: 196 tiles 84 us, now 5.)
__global__ __launch_bounds__(kWave * kColWaves) void colcarry_kernel(int p, int ntiles, const uint8_t *tile_carry,
                                                                     const int32_t *lasthead, const double *taila,
                                                                     const double *aggb, double *carry)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int j = __builtin_amdgcn_readfirstlane(blockIdx.x * kColWaves + threadIdx.x / kWave);
    if (j >= p) return;
    if (lane == 0) carry[j] = 0.0;
    double c = 0.0;   // S' entering the chunk's first tile
    for (int base = 0; base + 1 < ntiles; base += kWave) {
        const int t = base + lane;
        AffE e = AffOp::id();
        if (t + 1 < ntiles) {
            e = AffE{1u, 0.0, 0.0};
            if (tile_carry[t + 1]) e = AffE{lasthead[t] >= 0 ? 1u : 0u, taila[t], aggb[(int64_t)t * p + j]};
        }
        const AffE inc = wave_scan_e<AffOp>(e);
        const double out = inc.f ? inc.b : fma(inc.a, c, inc.b);
        if (t + 1 < ntiles) carry[(int64_t)(t + 1) * p + j] = out;
        c = readlane63(out);
    }
}

// kColBlock columns per wave: the row vectors (alpha, u, b, zq, row words,
// group indices) are loaded once per chunk for all of them, and the
// column-independent parts (flags, products of alpha) of the wave scan are
// formed once.
constexpr int kColBlock = 4;

// One DPP step of the shared-multiplier scan: every column's b uses the same
// (f, a) of the element it extends.
template <int CTRL, int ROWS, int CB>
__device__ __forceinline__ void aff_step(uint32_t &f, double &a, double (&b)[CB])
{
    const uint32_t sf = dpp_keep_u32<CTRL, ROWS>(0u, f);
    const double sa = dpp_keep<CTRL, ROWS>(1.0, a);
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        const double sb = dpp_keep<CTRL, ROWS>(0.0, b[c]);
        b[c] = f ? b[c] : fma(a, sb, b[c]);
    }
    a = f ? a : sa * a;
    f = f | sf;
}

// EFRON: at the end of a group with two or more events S1' goes to s1me (its rows of Z
// are formed with E1 by efron_z_kernel); the other groups' rows are the plain ones.
template <typename ZT, bool XBAR, bool EFRON>
__global__ __launch_bounds__(kWave * kColWaves) void colpass_kernel(const double *x, int64_t ld, int p, int64_t tile,
                                                                    int ntiles, const double *alpha, const double *u,
                                                                    const double *zq, const double *b,
                                                                    const uint32_t *meta, const int32_t *gidx,
                                                                    const uint8_t *tile_carry, const double *carry,
                                                                    int64_t ldz, const float *zscale, ZT *z, double *part,
                                                                    const int32_t *gidx2, double *s1me)
{
    constexpr int CB = kColBlock;
    const int lane = threadIdx.x & (kWave - 1);
    // XCD-aware order: workgroups are dealt to the 8 XCDs in turn, so workgroup
    // wg runs on XCD wg % 8; every column group of a tile goes to one XCD, whose
    // L2 then holds that tile's row vectors for all of its columns
    const int per_wg = kColWaves * CB;
    const int cgroups = (p + per_wg - 1) / per_wg;
    const int wg = blockIdx.x, xcd = wg & 7, k = wg >> 3;
    const int t = (k / cgroups) * 8 + xcd;
    const int j0 = __builtin_amdgcn_readfirstlane((k % cgroups) * per_wg + (int)(threadIdx.x / kWave) * CB);
    if (t >= ntiles || j0 >= p) return;   // whole wave; no workgroup barrier below
    const int64_t r_begin = (int64_t)t * tile, r_end = r_begin + tile;
    const double *xc[CB];
    bool live[CB];
    float zs[CB];
    double g[CB], d1[CB], d2[CB], cb[CB];   // cb: S'_j entering the chunk
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        const int j = j0 + c;
        live[c] = j < p;
        xc[c] = x + (int64_t)(live[c] ? j : j0) * ld;
        zs[c] = (zscale && live[c]) ? 1.0f / zscale[j] : 1.0f;
        g[c] = d1[c] = d2[c] = 0.0;
        cb[c] = (XBAR && live[c] && tile_carry[t]) ? carry[(int64_t)t * p + j] : 0.0;
    }
    // one chunk's loads: 4 consecutive rows per lane (16-byte loads); the next
    // chunk's loads are issued before this chunk is processed
    struct Chunk {
        double xv[CB][kColIpt], bv[kColIpt], av[kColIpt], uv[kColIpt], qv[kColIpt];
        uint32_t m[kColIpt];
        int32_t gi[kColIpt], g2[EFRON ? kColIpt : 1];
    };
    auto load_chunk = [&](Chunk &k, int64_t r0) {
#pragma unroll
        for (int c = 0; c < CB; ++c) load4(xc[c] + r0, k.xv[c]);
        load4(b + r0, k.bv);
        const uint4 mm = *reinterpret_cast<const uint4 *>(meta + r0);
        k.m[0] = mm.x;
        k.m[1] = mm.y;
        k.m[2] = mm.z;
        k.m[3] = mm.w;
        if (XBAR) {
            load4(alpha + r0, k.av);
            load4(u + r0, k.uv);
            load4(zq + r0, k.qv);
            const int4 gg = *reinterpret_cast<const int4 *>(gidx + r0);
            k.gi[0] = gg.x;
            k.gi[1] = gg.y;
            k.gi[2] = gg.z;
            k.gi[3] = gg.w;
            if constexpr (EFRON) {
                const int4 g2 = *reinterpret_cast<const int4 *>(gidx2 + r0);
                k.g2[0] = g2.x;
                k.g2[1] = g2.y;
                k.g2[2] = g2.z;
                k.g2[3] = g2.w;
            }
        }
    };
    Chunk cur;
    load_chunk(cur, r_begin + (int64_t)lane * kColIpt);
    for (int64_t base = r_begin; base < r_end; base += kColChunk) {
        Chunk nxt;
        const bool more = base + kColChunk < r_end;
        if (more) load_chunk(nxt, base + kColChunk + (int64_t)lane * kColIpt);
        double(&xv)[CB][kColIpt] = cur.xv;
        double(&bv)[kColIpt] = cur.bv;
        double(&av)[kColIpt] = cur.av;
        double(&uv)[kColIpt] = cur.uv;
        double(&qv)[kColIpt] = cur.qv;
        uint32_t(&m)[kColIpt] = cur.m;
        int32_t(&gi)[kColIpt] = cur.gi;
#pragma unroll
        for (int c = 0; c < CB; ++c) {
#pragma unroll
            for (int i = 0; i < kColIpt; ++i) {
                const double aw = bv[i] - ((m[i] & kEventBit) ? 1.0 : 0.0);   // w Lambda - delta
                g[c] = fma(xv[c][i], aw, g[c]);
                d1[c] = fma(xv[c][i] * xv[c][i], bv[i], d1[c]);
            }
        }
        if (XBAR) {
            // this lane's 4 rows folded: flags, product of alphas, and per column the map's offset
            uint32_t f = 0u;
            double a = 1.0, bb[CB];
#pragma unroll
            for (int c = 0; c < CB; ++c) bb[c] = 0.0;
#pragma unroll
            for (int i = 0; i < kColIpt; ++i) {
                const uint32_t fi = m[i] >> 31;
#pragma unroll
                for (int c = 0; c < CB; ++c) bb[c] = fi ? uv[i] * xv[c][i] : fma(av[i], bb[c], uv[i] * xv[c][i]);
                a = fi ? av[i] : a * av[i];
                f |= fi;
            }
            // inclusive scan across the wave
            aff_step<0x111, 0xF, CB>(f, a, bb);
            aff_step<0x112, 0xF, CB>(f, a, bb);
            aff_step<0x114, 0xF, CB>(f, a, bb);
            aff_step<0x118, 0xF, CB>(f, a, bb);
            aff_step<0x142, 0xA, CB>(f, a, bb);
            aff_step<0x143, 0xC, CB>(f, a, bb);
            // exclusive prefix of this lane = the inclusive value of lane - 1
            const uint32_t ef = dpp_keep_u32<0x138, 0xF>(0u, f);
            const double ea = dpp_keep<0x138, 0xF>(1.0, a);
            const uint32_t tf = (uint32_t)__builtin_amdgcn_readlane((int)f, 63);
            const double ta = readlane63(a);
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                const double eb = dpp_keep<0x138, 0xF>(0.0, bb[c]);
                double run = ef ? eb : fma(ea, cb[c], eb);   // S' entering this lane's first row
#pragma unroll
                for (int i = 0; i < kColIpt; ++i) {
                    const double ux = uv[i] * xv[c][i];
                    run = (m[i] >> 31) ? ux : fma(av[i], run, ux);
                    if ((m[i] & kCountMask) && live[c]) {
                        if (EFRON && cur.g2[EFRON ? i : 0] >= 0) {
                            s1me[(int64_t)cur.g2[EFRON ? i : 0] * p + j0 + c] = run;
                        } else {
                            const double zv = run * qv[i];   // sqrt(d) xbar
                            d2[c] = fma(zv, zv, d2[c]);
                            store_z<ZT>(&z[(int64_t)(j0 + c) * ldz + gi[i]], zv, zs[c]);
                        }
                    }
                }
                const double tb = readlane63(bb[c]);
                cb[c] = tf ? tb : fma(ta, cb[c], tb);
            }
        }
        if (more) cur = nxt;
    }
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        double gc = g[c], s1 = d1[c], s2 = d2[c];
        for (int off = 32; off >= 1; off >>= 1) {
            gc += __shfl_xor(gc, off, kWave);
            s1 += __shfl_xor(s1, off, kWave);
            s2 += __shfl_xor(s2, off, kWave);
        }
        if (lane == 0 && live[c]) {
            double *o = part + ((int64_t)t * p + j0 + c) * 3;
            o[0] = gc;
            o[1] = s1;
            o[2] = s2;
        }
    }
}

// Rows of Z of the multi-event groups (Efron): for group k and column j = blockIdx.y,
// E1' = sum over its event rows of exp(eta_r - m_end) x_rj, then z1 = l11 S1' + l21 E1' at the
// group's own row and z2 = l22 E1' at row n_groups + k; the workgroup's sum of z1^2 + z2^2 goes
// to epart[j][blockIdx.x] (fixed-order tree).
template <typename ZT>
__global__ __launch_bounds__(kRowBlock) void efron_z_kernel(const double *x, int64_t ld, int p, const int32_t *me_ptr,
                                                            const int32_t *me_row, const int32_t *me_end,
                                                            const double *me_w, const double *s1me,
                                                            const double *zq, const double *zq2, const double *zq3,
                                                            const int32_t *gidx, int64_t n_groups, int64_t n_multi,
                                                            int64_t ldz, const float *zscale, ZT *z, double *epart,
                                                            int eblocks)
{
    __shared__ double tree[kRowBlock];
    const int j = blockIdx.y;
    const int64_t k = (int64_t)blockIdx.x * kRowBlock + threadIdx.x;
    double sq = 0.0;
    if (k < n_multi && j < p) {
        const double *xj = x + (int64_t)j * ld;
        double e1 = 0.0;
        for (int32_t q = me_ptr[k]; q < me_ptr[k + 1]; ++q) e1 = fma(me_w[q], xj[me_row[q]], e1);
        const int32_t e = me_end[k];
        const double s1 = s1me[k * p + j];
        const double z1 = fma(zq[e], s1, zq2[e] * e1), z2 = zq3[e] * e1;
        const float inv = zscale ? 1.0f / zscale[j] : 1.0f;
        store_z<ZT>(&z[(int64_t)j * ldz + gidx[e]], z1, inv);
        store_z<ZT>(&z[(int64_t)j * ldz + n_groups + k], z2, inv);
        sq = fma(z1, z1, z2 * z2);
    }
    tree[threadIdx.x] = sq;
    __syncthreads();
    for (int h = kRowBlock / 2; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) tree[threadIdx.x] += tree[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0 && j < p) epart[(int64_t)j * eblocks + blockIdx.x] = tree[0];
}

// diag2[j] += the multi-event groups' parts, summed in block order
__global__ __launch_bounds__(kWave) void efron_d2_kernel(const double *epart, int eblocks, int p, double *diag2,
                                                         double *hdiag2)
{
    const int j = blockIdx.x * kWave + threadIdx.x;
    if (j < p) {
        double s = 0.0;
        for (int k = 0; k < eblocks; ++k) s += epart[(int64_t)j * eblocks + k];
        diag2[j] += s;
        hdiag2[j] = diag2[j];
    }
}

// Fixed-order sums over tiles: grad[j], diag1[j], diag2[j] (thread k sums
// tiles k, k + 256, ... in order, then a fixed-order tree over the threads);
// workgroup p sums the objective parts.
__device__ __forceinline__ double tree_sum_256(double v, double *red)
{
    red[threadIdx.x] = v;
    __syncthreads();
    for (int h = 128; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

__global__ __launch_bounds__(kRowBlock) void colreduce_kernel(const double *part, int p, int ntiles, double *grad,
                                                              double *diag1, double *diag2, const double *blockobj,
                                                              int nb, double *scal, const unsigned *flags,
                                                              double *hgrad, double *hscal, unsigned *hflags)
{
    __shared__ double red[kRowBlock / kWave];
    __shared__ double tree[256];
    const int j = blockIdx.x;
    if (j < p) {
        double sg = 0.0, s1 = 0.0, s2 = 0.0;
        for (int t = threadIdx.x; t < ntiles; t += kRowBlock) {
            const double *o = part + ((int64_t)t * p + j) * 3;
            sg += o[0];
            s1 += o[1];
            s2 += o[2];
        }
        sg = tree_sum_256(sg, tree);
        s1 = tree_sum_256(s1, tree);
        s2 = tree_sum_256(s2, tree);
        if (threadIdx.x == 0) {
            grad[j] = sg;
            diag1[j] = s1;
            diag2[j] = s2;
            hgrad[j] = sg;
            hgrad[p + j] = s1;
            hgrad[2 * p + j] = s2;
        }
    } else {
        double o = 0.0;
        for (int i = threadIdx.x; i < nb; i += kRowBlock) o += blockobj[i];
        o = block_sum(o, red);
        if (threadIdx.x == 0) {
            scal[1] = o;
            hscal[1] = o;
            *hflags = *flags;
        }
    }
}

// ------------------------------------------------------------------ row scans
//
// Segmented scans over all ld rows in tiles of `tile` rows: (1) each workgroup
// folds its tile into one aggregate, (2) one workgroup scans the aggregates
// into the value entering every tile, (3) each workgroup rescans its tile from
// there.  The element type and its operator come from affscan.hpp; a loader
// gives the element at scan position k and a writer stores the inclusive value.

constexpr int kScanThreads = 256, kScanWaves = kScanThreads / kWave;

template <class Op, class Ld, int PER>
__global__ __launch_bounds__(kScanThreads) void tscan_agg_kernel(Ld ldr, int64_t tile, typename Op::E *agg)
{
    using E = typename Op::E;
    __shared__ E wtot[kScanWaves];
    const int t = blockIdx.x;
    const int64_t per = PER > 0 ? PER : tile / kScanThreads;
    const int64_t k0 = (int64_t)t * tile + (int64_t)threadIdx.x * per;
    E f = Op::id();
    if constexpr (PER > 0) {
        E v[PER];   // all of the thread's rows in flight at once, in ascending address order
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int i = Ld::kReverse ? PER - 1 - q : q;
            v[i] = ldr(k0 + i);
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) f = Op::combine(f, v[i]);
    } else {
        for (int64_t i = 0; i < per; ++i) f = Op::combine(f, ldr(k0 + i));
    }
    E total;
    (void)block_exclusive_e<Op, kScanWaves>(f, wtot, total);
    if (threadIdx.x == 0) agg[t] = total;
}

template <class Op>
__global__ __launch_bounds__(1024) void tscan_carry_kernel(const typename Op::E *agg, int ntiles,
                                                           typename Op::E *carry)
{
    using E = typename Op::E;
    __shared__ E wtot[1024 / kWave];
    const int per = (ntiles + 1023) / 1024;
    const int t0 = threadIdx.x * per;
    E f = Op::id();
    for (int i = 0; i < per; ++i)
        if (t0 + i < ntiles) f = Op::combine(f, agg[t0 + i]);
    E total;
    E run = block_exclusive_e<Op, 1024 / kWave>(f, wtot, total);
    for (int i = 0; i < per; ++i) {
        const int t = t0 + i;
        if (t < ntiles) {
            carry[t] = run;
            run = Op::combine(run, agg[t]);
        }
    }
}

template <class Op, class Ld, class Wr, int PER>
__global__ __launch_bounds__(kScanThreads) void tscan_apply_kernel(Ld ldr, Wr wr, int64_t tile,
                                                                   const typename Op::E *carry)
{
    using E = typename Op::E;
    __shared__ E wtot[kScanWaves];
    const int t = blockIdx.x;
    const int64_t per = PER > 0 ? PER : tile / kScanThreads;
    const int64_t k0 = (int64_t)t * tile + (int64_t)threadIdx.x * per;
    if constexpr (PER > 0) {
        E v[PER];   // the thread's rows, loaded once, all in flight at once, in ascending address order
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int i = Ld::kReverse ? PER - 1 - q : q;
            v[i] = ldr(k0 + i);
        }
        E f = Op::id();
#pragma unroll
        for (int i = 0; i < PER; ++i) f = Op::combine(f, v[i]);
        E total;
        const E exc = block_exclusive_e<Op, kScanWaves>(f, wtot, total);
        E run = Op::combine(carry[t], exc);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            run = Op::combine(run, v[i]);
            wr(k0 + i, run);
        }
    } else {
        E f = Op::id();
        for (int64_t i = 0; i < per; ++i) f = Op::combine(f, ldr(k0 + i));
        E total;
        const E exc = block_exclusive_e<Op, kScanWaves>(f, wtot, total);
        E run = Op::combine(carry[t], exc);
        for (int64_t i = 0; i < per; ++i) {
            run = Op::combine(run, ldr(k0 + i));
            wr(k0 + i, run);
        }
    }
}

// running maximum of eta within each stratum (forward)
struct MaxLoad {
    static constexpr bool kReverse = false;   // scan position k is row k
    const double *eta;
    const uint32_t *meta;
    __device__ MaxE operator()(int64_t k) const { return MaxE{(meta[k] & kHeadBit) ? 1u : 0u, eta[k]}; }
};
struct MaxWrite {
    double *m;
    __device__ void operator()(int64_t k, const MaxE &e) const { m[k] = e.m; }
};

// S0' (forward): S0'_r = alpha_r S0'_{r-1} + u_r
struct S0Load {
    static constexpr bool kReverse = false;
    const double *alpha, *u;
    const uint32_t *meta;
    __device__ AffE operator()(int64_t k) const { return AffE{(meta[k] & kHeadBit) ? 1u : 0u, alpha[k], u[k]}; }
};
struct BWrite {
    double *out;
    __device__ void operator()(int64_t k, const AffE &e) const { out[k] = e.b; }
};

// Efron's E0' (forward): the running sum of u over event rows, restarting at stratum heads and
// after every row that ends a tie group with events, so at a group end it is the group's own
// E0 relative to exp(m_end): E0'_r = alpha_r E0'_{r-1} + delta_r u_r
struct E0Load {
    static constexpr bool kReverse = false;
    const double *alpha, *u;
    const uint32_t *meta;
    __device__ AffE operator()(int64_t k) const
    {
        const uint32_t mk = meta[k];
        const bool restart = (mk & kHeadBit) || k == 0 || (meta[k - 1] & kCountMask) != 0u;
        return AffE{restart ? 1u : 0u, alpha[k], (mk & kEventBit) ? u[k] : 0.0};
    }
};

// R (reverse, scan position k = row n-1-k): R_r = h'_r + alpha_{r+1} R_{r+1},
// a segment starting at each stratum's last row
struct RLoad {
    static constexpr bool kReverse = true;    // scan position k is row n - 1 - k
    const double *alpha, *h;
    const uint32_t *meta;
    int64_t n;
    __device__ AffE operator()(int64_t k) const
    {
        const int64_t r = n - 1 - k;
        const bool start = k == 0 || (meta[r + 1] & kHeadBit);
        return AffE{start ? 1u : 0u, start ? 1.0 : alpha[r + 1], h[r]};
    }
};
struct RWrite {
    double *out;
    int64_t n;
    __device__ void operator()(int64_t k, const AffE &e) const { out[n - 1 - k] = e.b; }
};

template <class Op, class Ld, class Wr>
int tile_scan(Ld ldr, Wr wr, int64_t n, int64_t tile, void *scratch, size_t scratch_bytes, hipStream_t stream)
{
    using E = typename Op::E;
    if (tile <= 0 || tile % kScanThreads != 0 || n % tile != 0) return -5;
    const int ntiles = (int)(n / tile);
    if (sizeof(E) * 2 * (size_t)ntiles > scratch_bytes) return -5;
    E *agg = static_cast<E *>(scratch);
    E *carry = agg + ntiles;
    // rows per thread as a compile-time count for the tile lengths of the layouts
    // (4096, 2048, 1024 and 512 rows), so that a thread's loads are all issued together
    const int64_t per = tile / kScanThreads;
#define COXMI_TSCAN(P)                                                                                     \
    do {                                                                                                   \
        tscan_agg_kernel<Op, Ld, P><<<ntiles, kScanThreads, 0, stream>>>(ldr, tile, agg);                 \
        tscan_carry_kernel<Op><<<1, 1024, 0, stream>>>(agg, ntiles, carry);                              \
        tscan_apply_kernel<Op, Ld, Wr, P><<<ntiles, kScanThreads, 0, stream>>>(ldr, wr, tile, carry);    \
    } while (0)
    if (per == 16) COXMI_TSCAN(16);
    else if (per == 8) COXMI_TSCAN(8);
    else if (per == 4) COXMI_TSCAN(4);
    else if (per == 2) COXMI_TSCAN(2);
    else COXMI_TSCAN(0);
#undef COXMI_TSCAN
    return hipGetLastError() == hipSuccess ? 0 : -3;
}

// ------------------------------------------------------------------ strata that fit a workgroup
//
// When every stratum has at most kSegRows rows, one workgroup evaluates whole strata at a time
// (a segment: consecutive strata of up to R rows) and nothing crosses workgroups: X beta of the
// segment's rows, the row scans, and the column sums, in one launch instead of about twenty.
//
//   1. X beta: a thread per row and column part, 8 columns in flight; the columns with beta_j != 0.
//   2. Row scans over the segment in registers and LDS (as the row-scan kernels below, one row
//      per thread).
//   3. Column sums: a wave takes 64 columns, a column per lane, and walks down the rows, so S1' is
//      a plain recurrence in a register and the three sums need no lane reductions (a wave of 64
//      rows per column spends four times the instructions on scan steps and reductions).  X comes in
//      8 rows at a time, two chunks ahead, coalesced along the rows, and turns through a wave-private LDS tile; the
//      row's factors are LDS broadcasts; xbar of the chunk's group ends goes back through the
//      tile and out along the groups.  With up to 512 columns spare waves take the segment's
//      strata in parts.
// X is read twice, at 5.3 TB/s (score only, N = 1e6, P = 200: 0.62 ms; X beta, three tiled row scans and the
// column pass took 0.71; with xbar in BF16 0.83 against 0.90; P = 500, N = 2.5e6: 4.4 against 5.1).
// Small data sets gain most, by the launches: N = 2e4, P = 20: 28 us against 53; N = 5e4, P = 300:
// 58 us against 156.
constexpr int kSegRows = 512, kSegThreads = 512, kSegWaves = kSegThreads / kWave;
constexpr int kSegChunk = 8, kSegTile = kSegChunk + 1;    // rows per chunk; padded LDS stride
constexpr int kSegGrid = 2 * kMaxGroups;                 // two workgroups per compute unit

__host__ __device__ __forceinline__ int seg_groups(int p) { return (p + kWave - 1) / kWave; }
__host__ __device__ __forceinline__ int seg_parts(int p)
{
    const int g = seg_groups(p);
    return g >= kSegWaves ? 1 : kSegWaves / g;
}

// Orders a wave's own LDS accesses across its lanes (they execute in order; this is for the compiler).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

size_t seg_lds_bytes(int p, int rows)
{
    return sizeof(double) * ((size_t)kSegWaves * kWave * kSegTile + 4 * ((size_t)rows + kSegChunk) +
                             3 * (size_t)seg_groups(p) * kWave * seg_parts(p) + (size_t)p) +
           sizeof(int) * (size_t)p;
}

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <typename ZT, bool XBAR>
__global__ __launch_bounds__(kSegThreads, 4) void strata_eval_kernel(const double *x, int64_t ld, int p,
                                                                  const double *beta, const uint32_t *meta,
                                                                  const EvalSeg *seg, int nseg, int wpp, double *bout,
                                                                  double *mout, double *rout, ZT *z, int64_t ldz,
                                                                  const float *zscale, double *part, double *blockobj,
                                                                  unsigned *flags)
{
    extern __shared__ double sm[];
    const int groups = seg_groups(p), parts = seg_parts(p);
    double *tiles = sm;                                                  // [waves][64][kSegTile]; scratch of phases 1, 2
    double2 *reca = reinterpret_cast<double2 *>(tiles + kSegWaves * kWave * kSegTile);   // alpha (0 at a head), u
    const int nrec = wpp * kWave + kSegChunk;
    double2 *recb = reca + nrec;                                         // b, zq
    double *acc = reinterpret_cast<double *>(recb + nrec);               // [groups * parts][3][64]
    double *bval = acc + 3 * groups * kWave * parts;                     // the nonzero beta_j
    int *bcol = reinterpret_cast<int *>(bval + p);
    __shared__ MaxE wm[kSegWaves];
    __shared__ AffE wf[kSegWaves], wb[kSegWaves];
    __shared__ unsigned long long headm[kSegWaves + 1], endm[kSegWaves + 1], evm[kSegWaves + 1];
    __shared__ double red[kSegWaves];
    __shared__ int s_nz;
    const int t = threadIdx.x, lane = t & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(t / kWave);

    for (int i = t; i < 3 * groups * kWave * parts; i += kSegThreads) acc[i] = 0.0;
    if (t < kSegChunk) {
        reca[wpp * kWave + t] = double2{0.0, 0.0};
        recb[wpp * kWave + t] = double2{0.0, 0.0};
    }
    if (t == 0) headm[kSegWaves] = endm[kSegWaves] = evm[kSegWaves] = 0ull;
    if (w == 0) {
        // the columns with beta_j != 0, in order
        int n = 0;
        for (int j0 = 0; j0 < p; j0 += kWave) {
            const double bj = j0 + lane < p ? beta[j0 + lane] : 0.0;
            const unsigned long long mask = __builtin_amdgcn_ballot_w64(bj != 0.0);
            if (bj != 0.0) {
                const int at = n + __popcll(mask & ((1ull << lane) - 1ull));
                bval[at] = bj;
                bcol[at] = j0 + lane;
            }
            n += __popcll(mask);
        }
        if (lane == 0) s_nz = n;
    }
    __syncthreads();
    const int nz = __builtin_amdgcn_readfirstlane(s_nz);
    const int np = kSegWaves / wpp;   // column parts of phase 1
    double obj = 0.0;

    for (int si = blockIdx.x; si < nseg; si += gridDim.x) {
        const int64_t row0 = __builtin_amdgcn_readfirstlane(seg[si].row0);
        const int n = __builtin_amdgcn_readfirstlane(seg[si].n), g0 = __builtin_amdgcn_readfirstlane(seg[si].g0);
        // ---- 1. X beta
        {
            const int q = w / wpp, r = (w % wpp) * kWave + lane;
            double e = 0.0;
            if (q < np && r < n) {
                const double *xr = x + row0 + r;
                const int k0 = (int)((int64_t)nz * q / np), k1 = (int)((int64_t)nz * (q + 1) / np);
                int k = k0;
                for (; k + 8 <= k1; k += 8) {
                    double v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = xr[(int64_t)__builtin_amdgcn_readfirstlane(bcol[k + i]) * ld];
#pragma unroll
                    for (int i = 0; i < 8; ++i) e = fma(v[i], bval[k + i], e);
                }
                for (; k < k1; ++k) e = fma(xr[(int64_t)__builtin_amdgcn_readfirstlane(bcol[k]) * ld], bval[k], e);
            }
            if (q < np) tiles[q * wpp * kWave + r] = e;
        }
        const bool in = t < n;
        const uint32_t mw = in ? meta[row0 + t] : kHeadBit;
        __syncthreads();
        // ---- 2. row scans
        {
            double e = 0.0;
            if (in)
                for (int q = 0; q < np; ++q) e += tiles[q * wpp * kWave + t];
            const uint32_t head = mw >> 31;
            const unsigned long long hm = __builtin_amdgcn_ballot_w64(in && head), em = __builtin_amdgcn_ballot_w64(in && (mw & kCountMask)),
                                     vm = __builtin_amdgcn_ballot_w64(in && (mw & kEventBit));
            if (lane == 0) {
                headm[w] = hm;
                endm[w] = em;
                evm[w] = vm;
            }
            MaxE mt;
            const MaxE me = {head, e};
            const MaxE mx = block_exclusive_e<MaxOp, kSegWaves>(me, wm, mt);
            const double m = MaxOp::combine(mx, me).m;
            const double alpha = head ? 1.0 : exp(mx.m - m), u = exp(e - m);
            AffE at;
            const AffE ae = {head, alpha, u};
            const double s0 = AffOp::combine(block_exclusive_e<AffOp, kSegWaves>(ae, wf, at), ae).b;
            const uint32_t d = mw & kCountMask;
            double hv = 0.0, zq = 0.0;
            if (d != 0u) {
                if (!(s0 >= 0.5) || !(s0 <= 1e300)) atomicOr(flags, 1u);
                hv = (double)d / s0;
                zq = hv / sqrt((double)d);
                obj += (double)d * (log(s0) + m);
            }
            if (mw & kEventBit) obj -= e;
            // reverse: thread t takes row n - 1 - t (every thread has passed the two scans' barriers, so
            // the sums of phase 1 are read)
            double *sh = tiles + kSegRows, *sa = tiles + 2 * kSegRows, *sr = tiles + 3 * kSegRows;
            if (in) {
                sh[t] = hv;
                sa[t] = alpha;
            }
            __syncthreads();
            const int r = n - 1 - t;
            AffE re = AffOp::id();
            if (r >= 0) {
                const bool start = r == n - 1 || ((headm[(r + 1) / kWave] >> ((r + 1) % kWave)) & 1ull);
                re = AffE{start ? 1u : 0u, start ? 1.0 : sa[r + 1], sh[r]};
            }
            AffE rt;
            const double R = AffOp::combine(block_exclusive_e<AffOp, kSegWaves>(re, wb, rt), re).b;
            if (r >= 0) sr[r] = R;
            __syncthreads();
            double b = 0.0;
            if (in) {
                b = u * sr[t];
                bout[row0 + t] = b;
                if (mout) {
                    mout[row0 + t] = m;
                    rout[row0 + t] = sr[t];
                }
            }
            if (t < wpp * kWave) {
                reca[t] = in ? double2{head ? 0.0 : alpha, u} : double2{0.0, 0.0};
                recb[t] = double2{b, zq};
            }
        }
        __syncthreads();
        // ---- 3. column sums
        auto bits = [&](const unsigned long long *mask, int r) {   // the 64 rows from r
            const int word = r / kWave, sft = r % kWave;
            const unsigned long long lo = mask[word] >> sft;
            return sft ? lo | (mask[word + 1 <= kSegWaves ? word + 1 : kSegWaves] << (kWave - sft)) : lo;
        };
        auto head_at = [&](int r) {   // the first head at or after row r, or n
            while (r < n) {
                const unsigned long long hm = bits(headm, r);
                if (hm) {
                    r += __builtin_ctzll(hm);
                    break;
                }
                r += kWave;
            }
            return r < n ? r : n;
        };
        for (int item = w; item < groups * parts; item += kSegWaves) {
            const int gi = item % groups, pi = item / groups;
            const int rs = __builtin_amdgcn_readfirstlane(pi == 0 ? 0 : head_at(n * pi / parts));
            const int re = __builtin_amdgcn_readfirstlane(pi == parts - 1 ? n : head_at(n * (pi + 1) / parts));
            if (rs >= re) continue;
            const int j0 = gi * kWave;
            int g = g0;   // the next group's index
            if (XBAR && rs > 0) {
                for (int k = 0; k < rs / kWave; ++k) g += __popcll(endm[k]);
                if (rs % kWave) g += __popcll(endm[rs / kWave] & ((1ull << (rs % kWave)) - 1ull));
                g = __builtin_amdgcn_readfirstlane(g);
            }
            double *tile = tiles + w * kWave * kSegTile;
            // loads: lane covers row lane % 8 of columns j0 + lane / 8 + 8 i (columns and rows beyond the
            // end are clamped, so that no load is conditional); sums: column j0 + lane
            const int lr = lane % kSegChunk, lc = lane / kSegChunk;
            uint32_t cl[kSegChunk];   // bytes from column j0 + 8 i (uniform) to this lane's
#pragma unroll
            for (int i = 0; i < kSegChunk; ++i) {
                const int most = p - 1 - (j0 + 8 * i);
                cl[i] = (uint32_t)(most <= 0 ? 0 : (lc < most ? lc : most)) * (uint32_t)ld * 8u;
            }
            const char *xg = reinterpret_cast<const char *>(x + (int64_t)j0 * ld + row0);
            auto load = [&](double (&v)[kSegChunk], int r) {
                const uint32_t at = (uint32_t)(r + lr < re ? r + lr : re - 1) * 8u;
#pragma unroll
                for (int i = 0; i < kSegChunk; ++i) {
                    const int ji = j0 + 8 * i < p ? 8 * i : p - 1 - j0;   // uniform
                    v[i] = *reinterpret_cast<const double *>(xg + (int64_t)ji * ld * 8 + (cl[i] + at));
                }
            };
            const float inv = (XBAR && zscale && j0 + lane < p) ? 1.0f / zscale[j0 + lane] : 1.0f;
            // Z as a buffer: stores beyond it are dropped, so none is conditional either (a conditional
            // store makes the next wait for X a wait for all stores).  FP64: these columns' [64][ldz].
            // BF16: blocks of 8 groups, [block][p][8] from the part's first block (see newton.h), so a
            // lane's 8 values are one 16-byte store and the wave's are contiguous; [p][ldz] here
            // meant runs of 16 bytes per column and line, written again and again (1.1 ms
            // instead of 0.6 at N = 1e6, P = 200).
            constexpr bool kBlocked = !std::is_same<ZT, double>::value;
            const int cols = p - j0 < kWave ? p - j0 : kWave;
            const int gfirst = g;
            __amdgpu_buffer_rsrc_t zbuf;
            if constexpr (kBlocked)
                zbuf = __builtin_amdgcn_make_buffer_rsrc(z + (int64_t)(gfirst / 8) * p * 8, (short)0,
                                                         (kSegRows / 8 + 1) * p * 16, kBufferWord3);
            else
                zbuf = __builtin_amdgcn_make_buffer_rsrc(XBAR ? z + (int64_t)j0 * ldz : z, (short)0,
                                                         XBAR ? (int)((uint32_t)cols * (uint32_t)ldz * 8u) : 0, kBufferWord3);
            const uint32_t zlane = lane < cols ? (uint32_t)(j0 + lane) * 16u : 0xfffffff0u;   // BF16: this lane's column
            u32x4 zreg = {0u, 0u, 0u, 0u}, zfull = {0u, 0u, 0u, 0u};   // the last 8 values; a completed block
            auto push = [&](uint32_t h) {
                zreg.x = __builtin_amdgcn_alignbit(zreg.y, zreg.x, 16);
                zreg.y = __builtin_amdgcn_alignbit(zreg.z, zreg.y, 16);
                zreg.z = __builtin_amdgcn_alignbit(zreg.w, zreg.z, 16);
                zreg.w = __builtin_amdgcn_alignbit(h, zreg.w, 16);
            };
            auto store_slots = [&](const u32x4 &v, int block, int q0, int q1) {   // an incomplete block
                for (int q = q0; q < q1; ++q) {
                    const uint32_t word = q < 4 ? (q < 2 ? v.x : v.y) : (q < 6 ? v.z : v.w);
                    const uint32_t off = zlane == 0xfffffff0u ? zlane : (uint32_t)block * (uint32_t)p * 16u + zlane + 2u * q;
                    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(q & 1 ? word >> 16 : word), zbuf, (int)off, 0, 0);
                }
            };
            double sg = 0.0, s1 = 0.0, s2 = 0.0, run = 0.0;
            double xa[kSegChunk], xb[kSegChunk];
            auto chunk = [&](double (&xr)[kSegChunk], int r) {
                const int left = re - r < kSegChunk ? re - r : kSegChunk;
                if (left < kSegChunk) {
#pragma unroll
                    for (int i = 0; i < kSegChunk; ++i) xr[i] = lr < left ? xr[i] : 0.0;
                }
#pragma unroll
                for (int i = 0; i < kSegChunk; ++i) tile[(lc + 8 * i) * kSegTile + lr] = xr[i];
                if (r + 2 * kSegChunk < re) load(xr, r + 2 * kSegChunk);
                wave_sync();
                const uint32_t live = (1u << left) - 1u;
                const uint32_t ends = __builtin_amdgcn_readfirstlane((uint32_t)bits(endm, r) & live);
                const uint32_t evs = __builtin_amdgcn_readfirstlane((uint32_t)bits(evm, r) & live);
                int k = 0;
                double *col = tile + lane * kSegTile;
#pragma unroll
                for (int i = 0; i < kSegChunk; ++i) {
                    const double xv = col[i];
                    const double2 cb = recb[r + i];
                    const double aw = cb.x - ((evs >> i) & 1u ? 1.0 : 0.0);   // w Lambda - delta
                    sg = fma(xv, aw, sg);
                    s1 = fma(xv * xv, cb.x, s1);
                    if constexpr (XBAR) {
                        const double2 ca = reca[r + i];
                        run = fma(ca.x, run, ca.y * xv);
                        if ((ends >> i) & 1u) {
                            const double zv = run * cb.y;   // sqrt(d) xbar
                            s2 = fma(zv, zv, s2);
                            if constexpr (kBlocked) {
                                const ZT h = __float2bfloat16((float)zv * inv);
                                push(__builtin_bit_cast(uint16_t, h));
                                ++g;
                                if ((g & 7) == 0) {   // at most once in 8 rows
                                    zfull = zreg;
                                    k = g / 8 - gfirst / 8;   // 1 + its block
                                }
                            } else {
                                col[k] = zv;   // slot k <= i of this lane's own row of the tile is already read
                                ++k;
                            }
                        }
                    }
                }
                if constexpr (XBAR && kBlocked) {
                    if (k == 1 && (gfirst & 7)) {   // the part's first block began in another part
                        store_slots(zfull, 0, gfirst & 7, 8);
                        k = 0;
                    }
                    const uint32_t off = k == 0 ? 0xfffffff0u : (uint32_t)(k - 1) * (uint32_t)p * 16u + zlane;
                    __builtin_amdgcn_raw_buffer_store_b128(zfull, zbuf, (int)(zlane == 0xfffffff0u ? zlane : off), 0, 0);
                } else if constexpr (XBAR) {
                    wave_sync();
#pragma unroll
                    for (int i = 0; i < kSegChunk; ++i) {
                        const long long slot = __double_as_longlong(tile[(lc + 8 * i) * kSegTile + lr]);
                        const uint32_t at = ((uint32_t)(lc + 8 * i) * (uint32_t)ldz + (uint32_t)(g + lr)) * 8u;
                        const u32x2 v = {(uint32_t)slot, (uint32_t)(slot >> 32)};
                        __builtin_amdgcn_raw_buffer_store_b64(v, zbuf, (int)(lr < k ? at : 0xfffffff0u), 0, 0);
                    }
                    g += k;
                }
                wave_sync();   // the tile is rewritten by the next chunk
            };
            load(xa, rs);
            if (rs + kSegChunk < re) load(xb, rs + kSegChunk);
            for (int r = rs; r < re; r += 2 * kSegChunk) {
                chunk(xa, r);
                if (r + kSegChunk < re) chunk(xb, r + kSegChunk);
            }
            if constexpr (XBAR && kBlocked) {
                if (g & 7) {
                    for (int q = g & 7; q < 8; ++q) push(0u);   // the block's values to their slots
                    store_slots(zreg, g / 8 - gfirst / 8, g / 8 == gfirst / 8 ? gfirst & 7 : 0, g & 7);
                }
            }
            double *o = acc + (size_t)item * 3 * kWave + lane;
            o[0] += sg;
            o[kWave] += s1;
            o[2 * kWave] += s2;
        }
        __syncthreads();   // the tiles are the next segment's scratch
    }
    for (int i = t; i < groups * parts * kWave; i += kSegThreads) {
        const int item = i / kWave, c = i % kWave, gi = item % groups, pi = item / groups, j = gi * kWave + c;
        if (j < p) {
            double *o = part + (((int64_t)blockIdx.x * parts + pi) * p + j) * 3;
            const double *v = acc + (size_t)item * 3 * kWave + c;
            o[0] = v[0];
            o[1] = v[kWave];
            o[2] = v[2 * kWave];
        }
    }
    obj = block_sum(obj, red);
    if (t == 0) blockobj[blockIdx.x] = obj;
}

}  // namespace

// ------------------------------------------------------------------ host launchers

constexpr size_t kSegMaxLds = 160 * 1024 - 2048;

// (64 columns of Z, ldz entries of at most 8 bytes each, are addressed by 32-bit offsets)
// (so are 8 columns of X, ld rows each)
bool segments_fit(int p, int64_t longest, int64_t ld, int64_t ldz)
{
    return ld < (int64_t)1 << 26 && longest <= kSegRows && seg_lds_bytes(p, kSegRows) <= kSegMaxLds && ldz < (int64_t)1 << 23;
}

// Rows of a segment: a power of two, at least the longest stratum.  Up to 512 rows while that is at
// most 64K entries of X, else 128 (measured, score only: P = 50, N = 1e6: 402, 261, 186, 180 us at
// 64 ... 512 rows; P = 200: 643, 602, 610, 684; P = 500, N = 2.5e6: 4.0, 3.3, 3.4, 3.6 ms; P = 1000:
// 3.1, 2.8, 3.2, 3.0); fewer where the data set would leave compute units idle.
int segment_rows(int64_t n, int p, int64_t longest)
{
    int R = kSegRows;
    while (R > 2 * kWave && (int64_t)R * p > 65536) R /= 2;
    while (R > kWave && (int64_t)R * kSegGrid > 2 * n) R /= 2;
    while (R < longest) R *= 2;
    return R;
}

int seg_round() { return kSegGrid; }
bool segment_may_grow(int rows, int p) { return 2 * rows <= kSegRows && (int64_t)2 * rows * p <= 66560; }

// The segments run kSegGrid at a time, one workgroup each, and a workgroup's time is the walk down the rows
// of its longest part (a stratum is never cut): where few strata fill a segment most of its waves
// stand idle, and tiles, which cut anywhere, win from a few columns on (N = 5e5, P = 20, strata of 350
// rows, score 116 us against 108, with xbar 213 against 126).  Microseconds of both, fitted to
// N = 2e3 ... 2e6, P = 5 ... 500, strata of 2 to 500 rows (within 13% and 9%); against the faster of the
// two on those the rule loses 3% on average.  Tiles grow with N, and beyond 2^20 rows (8192 to a tile) they
// lose to all segments but, with xbar, those of one long stratum each (N = 2e6, P = 20: strata of 20 rows
// 780 us against 355, of 256 rows 790 against 480, of 350 rows 700 against 750).  The widest sets of many
// rows come out even: N = 1e7, P = 500 in strata of 20 rows 15.2 to 16.7 ms against 15.4, of 64 rows 12.3
// against 15.1.
// FP64 Z is [p][ldz]: 64-byte runs per column, which the segments' waves write at once, so that beyond
// half a gigabyte of X (or 200 MB, with more than one segment per workgroup) the tiles' longer runs win
// (N = 1e6, P = 200: 1.02 ms against 1.40; N = 5e5, P = 64: 0.20 against 0.23).
bool segments_pay(int64_t n, int p, int64_t longest, int rows, int nseg, bool xbar, bool f64)
{
    const bool one_round = nseg <= kSegGrid;
    if (xbar && f64 && (double)n * p > (n > kSegGrid * (kSegRows / 2) && n <= 1 << 20 ? 2.4e7 : 6.4e7)) return false;
    if (n > 1 << 20) return !xbar || longest <= 300;
    const int groups = seg_groups(p), parts = seg_parts(p);
    const int strata = longest < rows ? rows / (int)longest : 1;   // of a segment
    const double part = (double)longest * ((strata + parts - 1) / parts) * ((groups * parts + kSegWaves - 1) / kSegWaves);
    const double mb = 8e-6 * (double)n * p, rounds = one_round ? 1.0 : std::ceil((double)nseg / kSegGrid);
    const double walk = rounds * (xbar ? (f64 ? 12.0 : 14.0) + 0.139 * part : 7.8 + 0.067 * part);
    const double bytes = mb * (xbar ? (f64 ? 0.78 : 0.50) : 0.36);
    // bound by reading X (and writing BF16 Z in its blocks), segments are the faster: BF16 fits of N = 1e6
    // in strata of 20 rows, P = 200: 10.35 ms against 11.38, P = 1000: 77.2 against 79.5
    if (!(xbar && f64) && !one_round && walk <= 0.6 * bytes) return true;
    const double segments = (xbar ? 17.0 : 16.5) + std::sqrt(walk * walk + bytes * bytes);
    const double tiles = xbar ? 49.0 + (f64 ? 0.50 : 0.43) * (mb + 1.4e-4 * (double)n) + 0.24 * p
                              : 47.0 + 0.33 * (mb + 1.6e-4 * (double)n) + 0.23 * p;
    return segments <= (one_round ? 1.15 : (xbar && f64 ? 0.95 : 1.0)) * tiles;
}

int seg_part_slots(int p, int nseg) { return (nseg < kSegGrid ? nseg : kSegGrid) * seg_parts(p); }

size_t rowscan_scratch_bytes(int ntiles) { return sizeof(AffE) * 2 * (size_t)ntiles + 256; }

int full_eval_launch(const FullEvalArgs &A, hipStream_t stream)
{
    const int64_t ld = A.ld;
    const int nb = (int)((ld + kRowBlock - 1) / kRowBlock);
    if (nb > A.max_blocks) return -5;
    hipError_t e = hipMemsetAsync(A.flags, 0, sizeof(unsigned), stream);
    if (e != hipSuccess) return -3;
    if (A.nseg > 0) {
        const int grid = A.nseg < kSegGrid ? A.nseg : kSegGrid;
        const int wpp = (A.seg_rows + kWave - 1) / kWave;
        const size_t lds = seg_lds_bytes(A.p, wpp * kWave);
        static LdsLimit limits[3];
        const void *fns[] = {reinterpret_cast<const void *>(&strata_eval_kernel<double, true>),
                             reinterpret_cast<const void *>(&strata_eval_kernel<__hip_bfloat16, true>),
                             reinterpret_cast<const void *>(&strata_eval_kernel<double, false>)};
        const int k = !A.want_xbar ? 2 : (A.ztype == kZF64 ? 0 : 1);
        if (limits[k].raise(fns[k], kSegMaxLds) != hipSuccess) return -3;
#define COXMI_SEGEVAL(ZT, XB)                                                                                     \
    strata_eval_kernel<ZT, XB><<<grid, kSegThreads, lds, stream>>>(                                               \
        A.x, ld, A.p, A.beta, A.meta, A.seg, A.nseg, wpp, A.b, A.want_rows ? A.m : nullptr,                       \
        A.want_rows ? A.lam : nullptr, static_cast<ZT *>(A.z), A.ldz, A.zscale, A.colpart, A.blockbuf, A.flags)
        if (!A.want_xbar) COXMI_SEGEVAL(double, false);
        else if (A.ztype == kZF64) COXMI_SEGEVAL(double, true);
        else COXMI_SEGEVAL(__hip_bfloat16, true);
#undef COXMI_SEGEVAL
        colreduce_kernel<<<A.p + 1, kRowBlock, 0, stream>>>(A.colpart, A.p, grid * seg_parts(A.p), A.grad, A.diag1,
                                                            A.diag2, A.blockbuf, grid, A.scal, A.flags, A.hgrad, A.hscal,
                                                            A.hflags);
        return hipGetLastError() == hipSuccess ? 0 : -3;
    }
    eta_kernel<<<nb, kRowBlock, 0, stream>>>(A.x, ld, A.p, A.beta, A.eta);
    int rc = tile_scan<MaxOp>(MaxLoad{A.eta, A.meta}, MaxWrite{A.m}, ld, A.tile, A.scan_scratch,
                              A.scan_scratch_bytes, stream);
    if (rc) return rc;
    prep_kernel<<<nb, kRowBlock, 0, stream>>>(A.eta, A.m, A.meta, ld, A.alpha, A.w);
    rc = tile_scan<AffOp>(S0Load{A.alpha, A.w, A.meta}, BWrite{A.s0}, ld, A.tile, A.scan_scratch,
                          A.scan_scratch_bytes, stream);
    if (rc) return rc;
    if (A.efron) {
        rc = tile_scan<AffOp>(E0Load{A.alpha, A.w, A.meta}, BWrite{A.e0}, ld, A.tile, A.scan_scratch,
                              A.scan_scratch_bytes, stream);
        if (rc) return rc;
        hazard_efron_kernel<<<nb, kRowBlock, 0, stream>>>(A.s0, A.e0, A.eta, A.m, A.meta, ld, A.h, A.kq, A.zq, A.zq2,
                                                          A.zq3, A.blockbuf, A.flags);
    } else {
        hazard_kernel<<<nb, kRowBlock, 0, stream>>>(A.s0, A.eta, A.m, A.meta, ld, A.h, A.zq, A.blockbuf, A.flags);
    }
    rc = tile_scan<AffOp>(RLoad{A.alpha, A.h, A.meta, ld}, RWrite{A.lam, ld}, ld, A.tile, A.scan_scratch,
                          A.scan_scratch_bytes, stream);
    if (rc) return rc;
    if (A.efron)
        rowweight_efron_kernel<<<nb, kRowBlock, 0, stream>>>(A.w, A.lam, A.eta, A.m, A.kq, A.gend, ld, A.b);
    else
        rowweight_kernel<<<nb, kRowBlock, 0, stream>>>(A.w, A.lam, ld, A.b);
    if (A.n_agg > 0) {
        double *wsuf = A.s0;   // read last by the hazards
        const int groups = (A.p + kAggCols - 1) / kAggCols;
        colweight_kernel<<<A.n_agg, kWeightBlock, 0, stream>>>(A.alpha, A.w, A.tile, A.agg_tiles, A.lasthead, wsuf,
                                                               A.agg + (int64_t)A.ntiles * A.p);
        colagg_kernel<<<(A.n_agg * groups + kColWaves - 1) / kColWaves, kWave * kColWaves, 0, stream>>>(
            A.x, ld, A.p, wsuf, A.tile, A.agg_tiles, A.n_agg, A.lasthead, A.agg);
        colcarry_kernel<<<(A.p + kColWaves - 1) / kColWaves, kWave * kColWaves, 0, stream>>>(
            A.p, A.ntiles, A.tile_carry, A.lasthead, A.agg + (int64_t)A.ntiles * A.p, A.agg, A.carry);
    }
    const int grid = 8 * ((A.ntiles + 7) / 8) * ((A.p + kColWaves * kColBlock - 1) / (kColWaves * kColBlock));
#define COXMI_COLPASS(ZT, XB, EF)                                                                              \
    colpass_kernel<ZT, XB, EF><<<grid, kWave * kColWaves, 0, stream>>>(                                        \
        A.x, ld, A.p, A.tile, A.ntiles, A.alpha, A.w, A.zq, A.b, A.meta, A.gidx, A.tile_carry, A.carry, A.ldz, \
        A.zscale, static_cast<ZT *>(A.z), A.colpart, A.gidx2, A.s1me)
    const bool ef = A.efron && A.n_multi > 0;
    if (!A.want_xbar) COXMI_COLPASS(double, false, false);
    else if (A.ztype == kZF64) {
        if (ef) COXMI_COLPASS(double, true, true);
        else COXMI_COLPASS(double, true, false);
    } else if (A.ztype == kZF32) {
        COXMI_COLPASS(float, true, false);
    } else {
        if (ef) COXMI_COLPASS(__hip_bfloat16, true, true);
        else COXMI_COLPASS(__hip_bfloat16, true, false);
    }
#undef COXMI_COLPASS
    colreduce_kernel<<<A.p + 1, kRowBlock, 0, stream>>>(A.colpart, A.p, A.ntiles, A.grad, A.diag1, A.diag2,
                                                        A.blockbuf, nb, A.scal, A.flags, A.hgrad, A.hscal, A.hflags);
    if (ef && A.want_xbar) {
        if (A.ztype == kZF32) return -5;
        efron_w_kernel<<<(unsigned)((A.n_multi + kRowBlock - 1) / kRowBlock), kRowBlock, 0, stream>>>(
            A.eta, A.m, A.me_ptr, A.me_row, A.me_end, A.n_multi, A.me_w);
        const dim3 zg((unsigned)A.eblocks, (unsigned)A.p);
        if (A.ztype == kZF64)
            efron_z_kernel<double><<<zg, kRowBlock, 0, stream>>>(
                A.x, ld, A.p, A.me_ptr, A.me_row, A.me_end, A.me_w, A.s1me, A.zq, A.zq2, A.zq3, A.gidx, A.n_groups,
                A.n_multi, A.ldz, A.zscale, static_cast<double *>(A.z), A.epart, A.eblocks);
        else
            efron_z_kernel<__hip_bfloat16><<<zg, kRowBlock, 0, stream>>>(
                A.x, ld, A.p, A.me_ptr, A.me_row, A.me_end, A.me_w, A.s1me, A.zq, A.zq2, A.zq3, A.gidx, A.n_groups,
                A.n_multi, A.ldz, A.zscale, static_cast<__hip_bfloat16 *>(A.z), A.epart, A.eblocks);
        efron_d2_kernel<<<(A.p + kWave - 1) / kWave, kWave, 0, stream>>>(A.epart, A.eblocks, A.p, A.diag2,
                                                                             A.hgrad + 2 * A.p);
    }
    e = hipGetLastError();
    return e == hipSuccess ? 0 : -3;
}

}  // namespace coxmi
