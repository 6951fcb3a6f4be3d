// ccd_kernel.hip -- persistent cyclic-coordinate-descent kernel for the stratified Cox model (gfx950).
//
// What one coordinate j computes (Sec. 2.7):
//   D = exp(X beta), N1 = X_j * D, N2 = X_j^2 * D            (Eqs. parallel_d, parallel_n1, parallel_n2)
//   segmented scans S[D], S[N1], S[N2] over the canonical rows  (Sec. 2.6)
//   g'  = -delta'X_j + delta'(S[N1]/S[D])                      (Eq. parallel_g)
//   g'' =  delta'(S[N2]/S[D]) - delta'(S[N1]/S[D])^2           (Eq. parallel_h)
//   Newton step with trust region and l1 rule                   (Sec. 2.4, Eq. newton)
//   X beta += X_j * step                                        (Eq. parallel_xb)
// Ties: an event reads the scans at the last row of its tie group; the row
// word carries d = number of events of the group on that row, so the
// reductions are sums over group ends of d * (...).
//
// How it maps onto the MI355X (our design, not the paper's):
//   * One persistent cooperative launch runs the whole fit.  Workgroup b of
//     BLOCK threads owns rows [b*BLOCK*IPT, (b+1)*BLOCK*IPT); each thread keeps
//     its IPT rows of X beta and of the row word in registers for the whole
//     fit, so a coordinate reads only x_j from HBM (8 B/row).  x_{j+1} is
//     loaded while coordinate j synchronises.
//   * Rows inside a workgroup: thread fold -> DPP wave scan -> LDS fold of the
//     wave totals.  A workgroup whose first row is not a stratum head takes
//     its carry from its predecessors' published tile aggregates (look-back,
//     one wave, 64 tiles per round).  When strata fit in a tile the host pads
//     the row layout so no stratum crosses a tile boundary, and the look-back
//     never runs.
//   * Per-coordinate sums are reduced per workgroup (DPP + LDS) and published
//     as epoch-tagged packets (two per workgroup, double-buffered by epoch
//     parity).  In every workgroup one wave gathers all of them -- up to four
//     workgroups' records per lane, all in flight at once -- reduces them in a
//     fixed order and takes the same scalar CCD step, which one barrier hands
//     to the other waves: one memory round trip after the last workgroup
//     publishes, everyone can move on.  Results are bit-reproducible.
//   * Data sets of up to 32 tiles run on one XCD: their packets then stay in its
//     L2 (an all-gather of 32 records takes 0.82 us, against 1.57 us for 20
//     workgroups across the chip and 2.27 us for 250).
//   * exp() uses one global shift c (within half a table step of the largest X beta
//     of the previous coordinate); ratios are shift-invariant and the objective adds c back.
//     A risk-set sum outside [1e-300, 1e300] stops the fit with a flag.
//
// What bounds it: the chain of one coordinate.  At N = 1e5, P = 1000, K = 5000 (49 tiles) a
// coordinate takes 3.7 us, of which the exchange is about 2; at N = 1e6, P = 50, K = 5e4
// (250 tiles) 5.65 us, of which the exchange is 2.5 and the passes 2.2 (16 row-waves per SIMD at
// about 45 instructions a row and 4 cycles each).  A SIMD issues one wave's 64 lanes in 4
// cycles, so what counts besides is instructions per wave: a lane step of the scans or sums
// costs the same with one row per thread as with eight, which is why tiles are few waves of
// several rows, the scans carry no flags (factors formed once per fit), and the LDS reads
// and dependent chains of a thread's rows are issued side by side.  Before these (512 threads
// of 1 row on all XCDs, flags in the scans, the table reads one after another, every
// thread folding the eight wave totals): 4.9 us and 6.7 us; N = 1e4 in 10 strata: 6.6 us, now 3.2.
#include <math.h>

#include <array>
#include <map>
#include <mutex>
#include <type_traits>

#include "internal.h"
#include "segscan.hpp"

namespace coxmi {

// Per-workgroup partial record.
struct Partial {
    double c1, c2, m2, obj;   // sums of d S1/S0, d (S2/S0 - (S1/S0)^2), d S2/S0; objective part
    uint32_t top;             // the largest X beta over real rows, as an unsigned key (see exp_rows)
    uint32_t err;             // a risk-set sum left the normal range
};

// Stop flags decided after a coordinate.
enum : uint32_t { kFlagNumeric = 1u, kFlagConverged = 2u, kFlagSweepLimit = 4u, kFlagAbort = 8u };

// What wave 0 hands to the other waves after a coordinate: one 16-byte LDS word.
struct alignas(16) StepWord {
    double step;
    uint32_t top;     // Partial::top over all workgroups
    uint32_t flags;
};

// A published record is 4 packet slots:
//   [0] (sum d S1/S0,              epoch, top)
//   [1] (sum d (S2/S0 - (S1/S0)^2), epoch, float(sum d S2/S0), NaN if a risk-set sum left range)
//   [2] (objective part,            epoch, 0)   -- only when the objective is wanted
//   [3] (sum d S2/S0,               epoch, 0)   -- only when evaluating (exact value for the caller)
// In a fit the side words only steer the shift and the degeneracy
// threshold, for which single precision is ample.
constexpr int kRecPackets = 4;

namespace {

size_t up256(size_t v) { return (v + 255) & ~size_t(255); }

}  // namespace

// Tile aggregates of the look-back: up to 6 packets per workgroup (Efron's scan element).
constexpr int kAggPackets = 6;

size_t sync_scratch_bytes(int grid)
{
    return up256(sizeof(SyncCtl)) + up256(sizeof(Packet) * kAggPackets * (size_t)grid) +
           up256(sizeof(Packet) * kRecPackets * 2 * (size_t)grid);
}

void carve_sync_scratch(void *base, int grid, CcdLaunch &L)
{
    char *c = static_cast<char *>(base);
    L.ctl = c;
    c += up256(sizeof(SyncCtl));
    L.agg = c;
    c += up256(sizeof(Packet) * kAggPackets * (size_t)grid);
    L.part = c;
    L.res = nullptr;
}

// ------------------------------------------------------------------ small helpers

// exp(x) by the table-driven method of Tang (ACM TOMS 15(2), 1989):
// x = (64 m + j) ln2/64 + r with |r| <= ln2/128, exp(x) = 2^m 2^(j/64) e^r, and
// e^r from its degree-5 Taylor polynomial (truncation below 2^-54 there).
// ln2/64 is split in two (the high part has 30 trailing zero bits, so n times
// it is exact) to form r without cancellation.  tab[j] = 2^(j/64), rounded
// to nearest, built on the host.  Accuracy about 1 ulp, like the libm exp.
//
// All rows of a thread go through each stage together: the indices and table reads of up to
// kExpGroup rows are issued before the first polynomial, so the LDS latency and the dependent
// FMA chains of different rows overlap (with two waves per SIMD there is little else to hide
// them; one row after another left pass 1 waiting on LDS).
constexpr int kExpGroup = 8;

//
// Returns the largest k of the rows: c + kmax ln2/64 is the largest X beta to within half a
// step of the table, which serves as the next coordinate's shift (any value near the maximum
// does) at half an integer instruction per row.  Published as kmax + kTopBias, an unsigned key
// whose identity is 0.
constexpr int kTopBias = 1 << 20;
constexpr double kTopStep = 0x1.62e42fefa39efp-7;   // ln2 / 64

template <int IPT>
__device__ __forceinline__ int exp_rows(double (&out)[IPT], const double (&eta)[IPT], double c, const double *tab)
{
    constexpr int GR = IPT < kExpGroup ? IPT : kExpGroup;
    int kmax = -kTopBias;
#pragma unroll
    for (int g = 0; g < IPT; g += GR) {
        double r[GR], t[GR];
        int k[GR];
#pragma unroll
        for (int i = 0; i < GR; ++i) {
            const double x = fmin(fmax(eta[g + i] - c, -746.0), 710.0);   // keeps k an int; results saturate to 0 / inf
            // n = rint(64 x / ln2): adding 1.5 * 2^52 leaves it in the low word, in two's complement
            const double m = fma(x, 0x1.71547652b82fep+6, 0x1.8p52);
            const double n = m - 0x1.8p52;
            k[i] = (int)(uint32_t)__double_as_longlong(m);
            t[i] = tab[k[i] & 63];
            r[i] = fma(-n, 0x1.62e42c0000000p-7, x);                     // ln2/64, high part
            r[i] = fma(-n, 0x1.f7d1cf79abc9ep-30, r[i]);                 // ln2/64, low part
        }
#pragma unroll
        for (int i = 0; i < GR; ++i) kmax = k[i] > kmax ? k[i] : kmax;
        __builtin_amdgcn_sched_barrier(0);
        double p[GR];
#pragma unroll
        for (int i = 0; i < GR; ++i) p[i] = fma(r[i], 1.0 / 120.0, 1.0 / 24.0);
#pragma unroll
        for (int i = 0; i < GR; ++i) p[i] = fma(r[i], p[i], 1.0 / 6.0);
#pragma unroll
        for (int i = 0; i < GR; ++i) p[i] = fma(r[i], p[i], 0.5);
#pragma unroll
        for (int i = 0; i < GR; ++i) p[i] = fma(r[i], p[i], 1.0);
#pragma unroll
        for (int i = 0; i < GR; ++i) p[i] = r[i] * p[i];
#pragma unroll
        for (int i = 0; i < GR; ++i) out[g + i] = ldexp(fma(t[i], p[i], t[i]), k[i] >> 6);
        __builtin_amdgcn_sched_barrier(0);
    }
    return kmax;
}

// Order-preserving unsigned key of a float (for the shift before any weight is known), and back.
__device__ __forceinline__ uint32_t float_key(float f)
{
    const uint32_t b = __float_as_uint(f);
    return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}
__device__ __forceinline__ float key_float(uint32_t k)
{
    return __uint_as_float(k ^ (~(uint32_t)((int32_t)k >> 31) | 0x80000000u));
}

// 1/a from the hardware estimate refined by two Newton steps (each squares
// the relative error), ending within about 1 ulp.
__device__ __forceinline__ double recip(double a)
{
    double r = __builtin_amdgcn_rcp(a);
    double e = fma(-a, r, 1.0);
    r = fma(r, e, r);
    e = fma(-a, r, 1.0);
    return fma(r, e, r);
}

template <int IPT>
__device__ __forceinline__ void load_rows(double (&v)[IPT], const double *p)
{
    if constexpr (IPT % 2 == 0) {
        const double2 *q = reinterpret_cast<const double2 *>(p);
#pragma unroll
        for (int i = 0; i < IPT / 2; ++i) {
            const double2 t = q[i];
            v[2 * i] = t.x;
            v[2 * i + 1] = t.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < IPT; ++i) v[i] = p[i];
    }
}

template <int IPT>
__device__ __forceinline__ void load_words(uint32_t (&v)[IPT], const uint32_t *p)
{
    if constexpr (IPT % 4 == 0) {
        const uint4 *q = reinterpret_cast<const uint4 *>(p);
#pragma unroll
        for (int i = 0; i < IPT / 4; ++i) {
            const uint4 t = q[i];
            v[4 * i] = t.x; v[4 * i + 1] = t.y; v[4 * i + 2] = t.z; v[4 * i + 3] = t.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < IPT; ++i) v[i] = p[i];
    }
}

// One column's values at a thread's IPT rows (XK, the kind of X).  Dense (0): IPT doubles
// from the column-major X.  Indicator (1): one bit per row, a thread's IPT bits in one unit
// (uint8 for IPT <= 8, uint16 for 16) at xbits[j * ldb + thread]; the value is 0.0 or 1.0,
// so every product formed with it equals the dense one exactly.  Sparse values (2): the
// same bits mark the nonzero rows, whose values lie in row order in xvals from xvoff[j];
// a wave's first one is at woff[j * nwaves + wave], a lane's after the nonzeros of the
// lanes below it (a prefix sum of bit counts across the wave) -- the values themselves,
// so every product again equals the dense one.
template <int IPT, int XK>
struct XCol;

template <int IPT>
struct XCol<IPT, 0> {
    double v[IPT];
    __device__ __forceinline__ void load(const CcdLaunch &L, int64_t ld, int64_t j, int64_t row0, int64_t)
    {
        load_rows<IPT>(v, L.x + j * ld + row0);
    }
    __device__ __forceinline__ double operator[](int i) const { return v[i]; }
};

template <int IPT>
struct XCol<IPT, 1> {
    using Unit = typename std::conditional<(IPT > 8), uint16_t, uint8_t>::type;
    uint32_t bits;
    __device__ __forceinline__ void load(const CcdLaunch &L, int64_t, int64_t j, int64_t, int64_t tg)
    {
        bits = static_cast<const Unit *>(L.xbits)[j * L.ldb + tg];
    }
    __device__ __forceinline__ double operator[](int i) const { return ((bits >> i) & 1u) ? 1.0 : 0.0; }
};

template <int IPT>
struct XCol<IPT, 2> {
    using Unit = typename std::conditional<(IPT > 8), uint16_t, uint8_t>::type;
    double v[IPT];
    // called by every lane of the wave (the prefix sum below is across the whole wave)
    __device__ __forceinline__ void load(const CcdLaunch &L, int64_t, int64_t j, int64_t, int64_t tg)
    {
        const uint32_t bits = static_cast<const Unit *>(L.xbits)[j * L.ldb + tg];
        const int lane = (int)(threadIdx.x & (kWave - 1));
        const int cnt = __popc(bits);
        int incl = cnt;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int up = __shfl_up(incl, d, kWave);
            if (lane >= d) incl += up;
        }
        const double *src = L.xvals + L.xvoff[j] + L.woff[j * L.nwaves + tg / kWave] + (incl - cnt);
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            const uint32_t below = bits & ((1u << i) - 1u);
            v[i] = ((bits >> i) & 1u) ? src[__popc(below)] : 0.0;
        }
    }
    __device__ __forceinline__ double operator[](int i) const { return v[i]; }
};

__device__ __forceinline__ Partial partial_identity()
{
    return Partial{0.0, 0.0, 0.0, 0.0, 0u, 0u};
}

// OBJ: the objective part takes part too (otherwise it is not touched).
template <bool OBJ>
__device__ __forceinline__ void partial_combine(Partial &a, const Partial &b)
{
    a.c1 += b.c1;
    a.c2 += b.c2;
    a.m2 += b.m2;
    if constexpr (OBJ) a.obj += b.obj;
    a.top = a.top > b.top ? a.top : b.top;
    a.err |= b.err;
}

template <int CTRL, int ROWS, bool OBJ>
__device__ __forceinline__ void dpp_step(Partial &x)
{
    Partial r = x;
    r.c1 = dpp_f64<CTRL, ROWS>(x.c1);
    r.c2 = dpp_f64<CTRL, ROWS>(x.c2);
    r.m2 = dpp_f64<CTRL, ROWS>(x.m2);
    if constexpr (OBJ) r.obj = dpp_f64<CTRL, ROWS>(x.obj);
    r.top = dpp_u32<CTRL, ROWS>(x.top);
    r.err = 0u;
    partial_combine<OBJ>(x, r);
}

// Wave reduction in a fixed lane order; the total ends in lane 63.
template <bool OBJ>
__device__ __forceinline__ void wave_reduce_partial(Partial &x)
{
    dpp_step<0x111, 0xF, OBJ>(x);
    dpp_step<0x112, 0xF, OBJ>(x);
    dpp_step<0x114, 0xF, OBJ>(x);
    dpp_step<0x118, 0xF, OBJ>(x);
    dpp_step<0x142, 0xA, OBJ>(x);
    dpp_step<0x143, 0xC, OBJ>(x);
    x.err = __builtin_amdgcn_ballot_w64(x.err != 0u) != 0 ? 1u : 0u;
}

// Workgroup reduction: every wave reduces its own rows, and after one barrier lane k of wave 0
// takes wave k's total and two or three more lane steps finish, so that the total is in lane NW - 1 of
// wave 0 -- the only wave that needs it (the others go on to wait for the step).  The wave
// totals stay in `red` until the barrier after the step.
template <int NW, bool OBJ>
__device__ __forceinline__ Partial block_reduce_partial(Partial x, Partial *red)
{
    static_assert(NW == 4 || NW == 8, "two or three lane steps");
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    wave_reduce_partial<OBJ>(x);
    if (lane == kWave - 1) red[w] = x;
    __syncthreads();
    if (w == 0) {
        x = red[lane & (NW - 1)];
        dpp_step<0x111, 0xF, OBJ>(x);
        dpp_step<0x112, 0xF, OBJ>(x);
        if constexpr (NW == 8) dpp_step<0x114, 0xF, OBJ>(x);
        x.err = (__builtin_amdgcn_ballot_w64(x.err != 0u) & ((1u << NW) - 1u)) != 0 ? 1u : 0u;
    }
    return x;
}

// Publish this workgroup's record for `epoch` (one lane); `extra` adds slots [2] and [3].
// local: every workgroup of the launch shares one L2 (see ccd_kernel).
__device__ __forceinline__ void publish_partial(const PacketArray &part, int G, int b, const Partial &x,
                                                uint32_t epoch, bool extra, bool local)
{
    const uint32_t slot = (uint32_t)(kRecPackets * ((epoch & 1u) * (uint32_t)G + (uint32_t)b));
    const float m2 = x.err ? __builtin_nanf("") : (float)fmin(x.m2, 3.0e38);
    packet_put(part, slot, x.c1, epoch, x.top, local);
    packet_put(part, slot + 1, x.c2, epoch, __float_as_uint(m2), local);
    if (extra) {
        packet_put(part, slot + 2, x.obj, epoch, 0u, local);
        packet_put(part, slot + 3, x.m2, epoch, 0u, local);
    }
}

// One CCD coordinate update (Sec. 2.4).  Newton step on the smooth part; with
// an l1 weight the step uses g' + gamma sgn(beta) away from 0, and at 0 the
// one-sided directional derivatives g' + gamma / g' - gamma pick the side (or
// no move).  The step is limited to the trust-region half-width, a step that
// would carry beta through 0 stops at 0, and the half-width becomes
// max(2 |step|, half-width / 2).  Columns with numerically zero curvature
// (g'' <= 1e-12 delta'(S[N2]/S[D])) do not move.
__device__ __forceinline__ double ccd_step(double beta, double g1, double g2, double m2, double gamma,
                                           double *trust, int *pinned)
{
    if (!(g2 > 1e-12 * fabs(m2)) || !isfinite(g2)) {
        *pinned = 1;
        return 0.0;
    }
    // the numerator of the Newton step (0: no move), then one division
    double num = g1;
    if (gamma > 0.0) {
        const double up = g1 + gamma, down = g1 - gamma;
        num = beta > 0.0 ? up : (beta < 0.0 ? down : (up < 0.0 ? up : (down > 0.0 ? down : 0.0)));
    }
    const double inv = recip(g2), q = num * inv;
    const double d = -fma(fma(-q, g2, num), inv, q);   // -num / g2, the quotient corrected once
    const double lim = *trust;
    double s = fabs(d) > lim ? lim : fabs(d);
    s = d < 0.0 ? -s : s;
    if (gamma > 0.0 && beta != 0.0) {
        const double nb = beta + s;
        if ((beta > 0.0 && nb < 0.0) || (beta < 0.0 && nb > 0.0)) s = -beta;
    }
    const double t2 = 2.0 * fabs(s), half = 0.5 * lim;
    *trust = t2 > half ? t2 : half;
    return s;
}

// One wave gathers the records of all G <= 64 PER workgroups for `epoch`: lane L
// waits for the records of workgroups L, L + 64, ... (every packet of
// every pending record in flight at once, re-polled together until all carry the
// epoch), folds them in that order, and the wave reduces the lane totals in a
// fixed DPP order -- so every workgroup obtains the same bits regardless of
// arrival times.  Every lane of the wave receives the total.  Returns false
// (uniformly) once a wait has timed out or another workgroup aborted.  Packets
// first .. first + NP - 1 of each record are polled.
template <int NP, int PER, bool SHORT>
__device__ __forceinline__ bool poll_records(const PacketArray &part, int G, uint32_t epoch, SyncCtl *ctl,
                                             u32x4 (&r)[PER][NP], int first = 0)
{
    const int lane = threadIdx.x & (kWave - 1);
    bool done[PER];
    uint32_t slot[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int q = lane + kWave * k;
        done[k] = q >= G;
        slot[k] = (uint32_t)(kRecPackets * ((epoch & 1u) * (uint32_t)G + (uint32_t)q) + first);
    }
    WaitBudget wb;
    bool ok = true;
    for (;;) {
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (!done[k])
#pragma unroll
                for (int pk = 0; pk < NP; ++pk) r[k][pk] = packet_get(part, slot[k] + pk);
        bool all = true;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (!done[k]) {
                bool fresh = true;
#pragma unroll
                for (int pk = 0; pk < NP; ++pk) fresh = fresh && r[k][pk].z == epoch;
                done[k] = fresh;
                all = all && fresh;
            }
        }
        if (all) break;
        if (!wb.keep_waiting<SHORT>(ctl)) {
            ok = false;
            break;
        }
    }
    return __builtin_amdgcn_ballot_w64(!ok) == 0;
}

template <int PER, bool SHORT>
__device__ __forceinline__ bool gather_records(const PacketArray &part, int G, uint32_t epoch, bool extra,
                                               SyncCtl *ctl, Partial &total)
{
    const int lane = threadIdx.x & (kWave - 1);
    Partial x = partial_identity();
    {
        u32x4 r[PER][2];
        if (!poll_records<2, PER, SHORT>(part, G, epoch, ctl, r)) return false;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (lane + kWave * k < G) {
                const float m2 = __uint_as_float(r[k][1].w);
                const Partial y = {packet_value(r[k][0]), packet_value(r[k][1]), (double)m2, 0.0,
                                   r[k][0].w, (m2 == m2) ? 0u : 1u};
                partial_combine<false>(x, y);
            }
        }
    }
    if (extra) {
        // the objective and the exact second moment (written with the two above): a second,
        // short poll on the first coordinate of a sweep and in evaluations only
        u32x4 r[PER][2];
        if (!poll_records<2, PER, SHORT>(part, G, epoch, ctl, r, 2)) return false;
        double obj = 0.0, m2 = 0.0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (lane + kWave * k < G) {
                obj += packet_value(r[k][0]);
                m2 += packet_value(r[k][1]);
            }
        }
        x.obj = obj;
        x.m2 = m2;
        wave_reduce_partial<true>(x);
    } else {
        wave_reduce_partial<false>(x);
    }
    total.c1 = lane63_f64(x.c1);
    total.c2 = lane63_f64(x.c2);
    total.m2 = lane63_f64(x.m2);
    total.obj = extra ? lane63_f64(x.obj) : 0.0;
    total.top = (uint32_t)__builtin_amdgcn_readlane((int)x.top, 63);
    total.err = x.err;
    return true;
}

// SHORT: how a wait for four records per lane is laid out (WaitBudget::keep_waiting).
template <bool SHORT>
__device__ __forceinline__ bool gather_wave(const PacketArray &part, int G, uint32_t epoch, bool extra, SyncCtl *ctl,
                                            Partial &total)
{
    if (G <= kWave) return gather_records<1, true>(part, G, epoch, extra, ctl, total);
    return gather_records<kMaxGroups / kWave, SHORT>(part, G, epoch, extra, ctl, total);
}

// Tie-group terms of one row, added to v (Sec. 2.4 derivatives).  S = (S0, S1, S2): the
// inclusive risk-set sums at the row; d: the events of the tie group ending at the row (0 when
// the row ends no group with events, and then nothing is added).
//   Breslow (the risk sets of Eq. strat_l taken literally): every tied event sees S,
//     so the group adds d S1/S0, d (S2/S0 - (S1/S0)^2), d S2/S0, d (log S0 + c).  Evaluated
//     on every row without branches (d = 0 adds zeros; S0 is replaced by 1 there so that
//     no infinity enters), in pass2 below.
//   Efron (1977): E = (E0, E1, E2), the same sums over the group's own events; the l-th
//     of its d events sees S - (l/d) E, l = 0..d-1 (d = 1 is Breslow's term exactly).
template <bool WANT_OBJ>
__device__ __forceinline__ void group_terms_efron(Partial &v, uint32_t d, const double (&S)[3], const double (&E)[3],
                                                  double c)
{
    const double s0 = S[0];
    if (d == 0u) return;
    if (!(s0 >= 1e-300) || !(s0 <= 1e300)) v.err = 1u;
    const double dd = (double)d;
    for (uint32_t l = 0; l < d; ++l) {
        const double a = (double)l / dd;
        const double A = s0 - a * E[0];
        const double inv = recip(A);
        const double r1 = (S[1] - a * E[1]) * inv, r2 = (S[2] - a * E[2]) * inv;
        v.c1 += r1;
        v.c2 += fma(-r1, r1, r2);   // one rounding whichever way r2 was formed (r2 = r1 on indicator X)
        v.m2 += r2;
        if constexpr (WANT_OBJ) v.obj += log(A) + c;
    }
}

// Scan element of one row.  Components 0..NC-1: (D, N1, N2) restarting at stratum heads
// (flag bit 0).  On indicator X (XK = 1) x^2 = x, so N2 is N1 exactly and is left out (NC = 2).
// Efron adds components NC..2 NC - 1: the same values on event rows only, restarting
// after every row that ends a tie group with events (flag bit 1; such a row contributes 0
// itself, so the running value before it plus its own values are its group's event sums).
// An event-free stretch adds nothing, so these sums need no restart at stratum heads.
template <int XK>
constexpr int kRowComp = XK == 1 ? 2 : 3;
template <bool EFRON, int XK>
using RowVal = SegVal<(EFRON ? 2 : 1) * kRowComp<XK>, kRowComp<XK>>;

template <bool EFRON, int XK>
__device__ __forceinline__ RowVal<EFRON, XK> row_value(uint32_t m, double w, double x)
{
    constexpr int NC = kRowComp<XK>;
    RowVal<EFRON, XK> r;
    r.f = m >> 31;
    r.v[0] = w;
    r.v[1] = x * w;
    if constexpr (NC == 3) r.v[2] = x * r.v[1];
    if constexpr (EFRON) {
        const bool end = (m & kCountMask) != 0u, ev = (m & kEventBit) != 0u;
        r.f |= end ? 2u : 0u;
        const bool keep = ev && !end;
#pragma unroll
        for (int k = 0; k < NC; ++k) r.v[NC + k] = keep ? r.v[k] : 0.0;
    }
    return r;
}

// 1.0 or 0.0 as the factor that keeps or drops what a scan carries in.
__device__ __forceinline__ double keep_factor(bool keep)
{
    return __longlong_as_double(keep ? 0x3ff0000000000000ll : 0ll);
}

// The sums of several rows' values without flags: the flags of every step of the scans are the
// same for every coordinate, so the factors that keep or drop the carried value are formed once
// per fit (Breslow; Efron's six components take the general operator of segscan.hpp).
template <int NC>
struct Vals {
    double v[NC];
};

template <int CTRL, int ROWS, int NC>
__device__ __forceinline__ Vals<NC> dpp_vals(const Vals<NC> &x)
{
    Vals<NC> r;
#pragma unroll
    for (int k = 0; k < NC; ++k) r.v[k] = dpp_f64<CTRL, ROWS>(x.v[k]);
    return r;
}

template <int NC>
__device__ __forceinline__ Vals<NC> add_kept(const Vals<NC> &a, double keep, const Vals<NC> &b)
{
    Vals<NC> r;
#pragma unroll
    for (int k = 0; k < NC; ++k) r.v[k] = fma(a.v[k], keep, b.v[k]);
    return r;
}

template <int NC>
__device__ __forceinline__ Vals<NC> lane_vals(const Vals<NC> &x, int src)
{
    Vals<NC> r;
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        const long long b = __double_as_longlong(x.v[k]);
        const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), src);
        const int hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
        r.v[k] = __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
    }
    return r;
}

// Factors of one thread's place in the scans.
template <int NW>
struct ScanKeep {
    double wave[6];      // the six lane steps of the wave scan
    double tot[3];       // the lane steps over the wave totals (lane k: wave k)
    double exc, carry;   // what the earlier waves, and the earlier tiles, add to this thread
    uint32_t tile_flag;  // the tile holds a head

    // f: the thread's rows hold a head.  Called by every thread; two barriers.
    __device__ __forceinline__ void init(uint32_t f, uint32_t *lds)
    {
        const int lane = threadIdx.x & (kWave - 1);
        const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
        wave[0] = keep_factor(f == 0u); f |= dpp_u32<0x111, 0xF>(f);
        wave[1] = keep_factor(f == 0u); f |= dpp_u32<0x112, 0xF>(f);
        wave[2] = keep_factor(f == 0u); f |= dpp_u32<0x114, 0xF>(f);
        wave[3] = keep_factor(f == 0u); f |= dpp_u32<0x118, 0xF>(f);
        wave[4] = keep_factor(f == 0u); f |= dpp_u32<0x142, 0xA>(f);
        wave[5] = keep_factor(f == 0u); f |= dpp_u32<0x143, 0xC>(f);
        const uint32_t before = dpp_u32<0x138, 0xF>(f);   // a head in the wave's rows before this thread's
        if (lane == kWave - 1) lds[w] = f;
        __syncthreads();
        uint32_t g = lds[lane & (NW - 1)];
        __syncthreads();
        tot[0] = keep_factor(g == 0u); g |= dpp_u32<0x111, 0xF>(g);
        tot[1] = keep_factor(g == 0u); g |= dpp_u32<0x112, 0xF>(g);
        tot[2] = keep_factor(g == 0u);
        if constexpr (NW == 8) g |= dpp_u32<0x114, 0xF>(g);
        tile_flag = (uint32_t)__builtin_amdgcn_readlane((int)g, NW - 1);
        const uint32_t earlier = w > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)g, w > 0 ? w - 1 : 0) : 0u;
        exc = keep_factor(w > 0 && before == 0u);
        carry = keep_factor((before | earlier) == 0u);
    }

    template <int NC>
    __device__ __forceinline__ Vals<NC> wave_scan(Vals<NC> x) const
    {
        x = add_kept(dpp_vals<0x111, 0xF>(x), wave[0], x);
        x = add_kept(dpp_vals<0x112, 0xF>(x), wave[1], x);
        x = add_kept(dpp_vals<0x114, 0xF>(x), wave[2], x);
        x = add_kept(dpp_vals<0x118, 0xF>(x), wave[3], x);
        x = add_kept(dpp_vals<0x142, 0xA>(x), wave[4], x);
        x = add_kept(dpp_vals<0x143, 0xC>(x), wave[5], x);
        return x;
    }

    // The workgroup's exclusive scan; `total` receives the tile's total.  One barrier.
    template <int NC>
    __device__ __forceinline__ Vals<NC> block_scan(const Vals<NC> &x, Vals<NC> *lds, Vals<NC> &total) const
    {
        const int lane = threadIdx.x & (kWave - 1);
        const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
        const Vals<NC> inc = wave_scan(x);
        if (lane == kWave - 1) lds[w] = inc;
        const Vals<NC> before = dpp_vals<0x138, 0xF>(inc);
        __syncthreads();
        Vals<NC> t = lds[lane & (NW - 1)];
        t = add_kept(dpp_vals<0x111, 0xF>(t), tot[0], t);
        t = add_kept(dpp_vals<0x112, 0xF>(t), tot[1], t);
        if constexpr (NW == 8) t = add_kept(dpp_vals<0x114, 0xF>(t), tot[2], t);
        total = lane_vals(t, NW - 1);
        return add_kept(lane_vals(t, w > 0 ? w - 1 : 0), exc, before);
    }
};

// Pass 2 over a thread's rows: the inclusive prefixes at group ends, the group-end terms, and
// (WANT_OBJ, the first coordinate of a sweep) the objective's parts.
//
// Breslow: the terms go through each stage for kTermGroup rows together, so that the
// reciprocals' dependent steps overlap.  A row that ends no group with events has d = 0; there
// the high word of S0 is replaced by 1.0's, which keeps the reciprocal finite.  The range test
// compares high words (S0 in [1e-300, 1e300] up to a relative 1e-6 at either end; a NaN or a
// negative value is out).
constexpr int kTermGroup = 4;
constexpr uint32_t kHiLow = 0x01a56e1fu, kHiHigh = 0x7e37e43cu, kHiOne = 0x3ff00000u;

// S(i, k): component k of the inclusive prefix at row i
template <int IPT, int NC, bool WANT_OBJ, class Prefix>
__device__ __forceinline__ void pass2_breslow(Partial &v, const uint32_t (&meta)[IPT], double c, Prefix S)
{
    constexpr int GR = IPT < kTermGroup ? IPT : kTermGroup;
    uint32_t lo = kHiOne, hi = kHiOne;
#pragma unroll
    for (int g = 0; g < IPT; g += GR) {
        double sg[GR], s1[GR], s2[GR], inv[GR];
#pragma unroll
        for (int i = 0; i < GR; ++i) {
            double row[NC];
            S(g + i, row);
            const long long b = __double_as_longlong(row[0]);
            const uint32_t h = (meta[g + i] & kCountMask) ? (uint32_t)(b >> 32) : kHiOne;
            lo = h < lo ? h : lo;
            hi = h > hi ? h : hi;
            sg[i] = __longlong_as_double((long long)(((unsigned long long)h << 32) | (uint32_t)b));
            s1[i] = row[1];
            s2[i] = row[NC - 1];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < GR; ++i) inv[i] = __builtin_amdgcn_rcp(sg[i]);
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            double e[GR];
#pragma unroll
            for (int i = 0; i < GR; ++i) e[i] = fma(-sg[i], inv[i], 1.0);
#pragma unroll
            for (int i = 0; i < GR; ++i) inv[i] = fma(inv[i], e[i], inv[i]);
        }
#pragma unroll
        for (int i = 0; i < GR; ++i) {
            const double dd = (double)(meta[g + i] & kCountMask);
            const double r1 = s1[i] * inv[i], r2 = NC == 2 ? r1 : s2[i] * inv[i];
            v.c1 = fma(dd, r1, v.c1);
            v.c2 = fma(dd, fma(-r1, r1, r2), v.c2);
            v.m2 = fma(dd, r2, v.m2);
            if constexpr (WANT_OBJ) v.obj = fma(dd, log(sg[i]) + c, v.obj);
        }
    }
    if (lo < kHiLow || hi > kHiHigh) v.err = 1u;
}

template <int IPT, int XK, bool WANT_OBJ>
__device__ __forceinline__ void pass2_efron(Partial &v, RowVal<true, XK> run, const uint32_t (&meta)[IPT],
                                            const double (&wv)[IPT], const XCol<IPT, XK> &xc, double c)
{
    constexpr int NC = kRowComp<XK>;
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const RowVal<true, XK> r = row_value<true, XK>(meta[i], wv[i], xc[i]);
        double E[3];
        // this row's group's event sums: the running value before it plus its own share
        const bool ev = (meta[i] & kEventBit) != 0u;
#pragma unroll
        for (int k = 0; k < NC; ++k) E[k] = run.v[NC + k] + (ev ? r.v[k] : 0.0);
        E[2] = E[NC - 1];
        run = seg_combine(run, r);
        const double S[3] = {run.v[0], run.v[1], run.v[NC - 1]};
        group_terms_efron<WANT_OBJ>(v, meta[i] & kCountMask, S, E, c);
    }
}

// ------------------------------------------------------------------ the persistent kernel

// WAVE: the layout puts every stratum inside one wave's rows, so a wave's first row is a
// stratum head and its scan needs nothing from the other waves: no workgroup scan, no barrier.
template <int BLOCK, int IPT, int XK, bool EFRON, bool WAVE>
__global__ __launch_bounds__(BLOCK) void ccd_kernel(CcdLaunch L)
{
    constexpr int NW = BLOCK / kWave;
    using RV = RowVal<EFRON, XK>;
    constexpr int NC = kRowComp<XK>, KV = (EFRON ? 2 : 1) * NC;
    // Breslow with up to 8 rows per thread keeps the rows' prefixes within the thread from pass 1
    // to pass 2 (one FMA per component adds the carry); 16 rows of them do not fit in registers
    constexpr bool KEEP = IPT <= 8;
    static_assert(BLOCK % kWave == 0 && (NW == 4 || NW == 8), "block shape");
    extern __shared__ double smem_dyn[];     // beta (the same in every workgroup)
    __shared__ RV s_wtot[EFRON ? NW : 1];
    __shared__ Vals<NC> s_vtot[NW];
    __shared__ Partial s_red[NW];        // this workgroup's own reduction
    __shared__ uint32_t s_flag[NW];
    __shared__ RV s_win[kMaxGroups / kWave];
    __shared__ int s_abort;
    __shared__ double s_exptab[64];
    __shared__ StepWord s_word;          // wave 0's step and shift for the next coordinate

    // One XCD: the launch has `spread` workgroups for each one that works, and workgroups go to
    // the XCDs in turn, so those that work share an L2.
    if (L.spread > 1 && blockIdx.x % L.spread != 0) return;
    const int p = L.p;
    const int G = gridDim.x / L.spread, b = blockIdx.x / L.spread, t = threadIdx.x;
    const int lane = t & (kWave - 1), w = t / kWave;
    const bool writer = (b == 0 && t == 0);   // writes the outputs
    SyncCtl *ctl = static_cast<SyncCtl *>(L.ctl);
    const PacketArray agg = packet_array(L.agg, sizeof(Packet) * KV * (size_t)G);
    const PacketArray part = packet_array(L.part, sizeof(Packet) * kRecPackets * 2 * (size_t)G);
    const int64_t ld = (int64_t)G * BLOCK * IPT;
    const int64_t tile0 = (int64_t)b * BLOCK * IPT;
    const int64_t row0 = tile0 + (int64_t)t * IPT;
    const int64_t tg = (int64_t)b * BLOCK + t;      // the thread's unit in an indicator column
    const bool fit = (L.mode == kModeFit);

    double *sbeta = smem_dyn;
    double *trust = L.trust + (int64_t)b * p;      // this workgroup's copy of the trust half-widths
    for (int j = t; j < p; j += BLOCK) {
        sbeta[j] = L.beta[j];
        trust[j] = 1.0;
    }
    if (t == 0) s_abort = 0;
    if (t < 64) s_exptab[t] = L.exp_tab[t];
    uint32_t meta[IPT];
    double eta[IPT];
    load_words<IPT>(meta, L.meta + row0);
#pragma unroll
    for (int i = 0; i < IPT; ++i) eta[i] = (meta[i] & kPadBit) ? -INFINITY : 0.0;   // padding: weight 0, never the maximum
    const bool tile_head = (L.meta[tile0] & kHeadBit) != 0u;
    ScanKeep<NW> keep;
    double krow[IPT], kall[IPT];   // a row keeps the row before it; its prefix keeps what enters the thread
    {
        uint32_t f = 0u;
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            f |= meta[i] >> 31;
            krow[i] = keep_factor(!(meta[i] & kHeadBit));
            kall[i] = keep_factor(f == 0u);
        }
        if constexpr (!EFRON) keep.init(f, s_flag);
    }

    // X beta0 (columns with beta0_j = 0 are skipped)
    for (int j = 0; j < p; ++j) {
        const double bj = L.beta[j];
        if (bj != 0.0) {
            XCol<IPT, XK> xv;
            xv.load(L, ld, j, row0, tg);
#pragma unroll
            for (int i = 0; i < IPT; ++i) eta[i] = fma(xv[i], bj, eta[i]);
        }
    }
    __syncthreads();

    // epoch 1: the initial shift, the largest X beta over the real rows, and with `spread` the
    // XCDs the working workgroups run on (c1, c2: sums of the id and of its square, so that
    // G c2 = c1^2 exactly when all are equal).  Packets of one XCD can stay in its L2; if the
    // workgroups turn out to be spread after all, they go through to device memory as always.
    uint32_t epoch = 1;
    double c;
    bool local = false;
    {
        Partial v = partial_identity();
        float most = -INFINITY;   // fmaxf passes a NaN by: its row has no weight either (as a key it would be the largest)
#pragma unroll
        for (int i = 0; i < IPT; ++i) most = fmaxf(most, (float)eta[i]);   // -INFINITY at padding
        v.top = float_key(most);
        v = block_reduce_partial<NW, false>(v, s_red);
        if (w == 0) {
            const double xcc = (double)xcc_id();
            v.c1 = xcc;
            v.c2 = xcc * xcc;
            if (lane == NW - 1) publish_partial(part, G, b, v, epoch, false, false);
            Partial tot;
            const bool ok = gather_wave<!WAVE>(part, G, epoch, false, ctl, tot);
            if (lane == 0) {
                const bool one = ok && (G == 1 || (L.spread > 1 && (double)G * tot.c2 == tot.c1 * tot.c1));
                s_word = StepWord{one ? 1.0 : 0.0, ok ? tot.top : 0u, ok ? 0u : (uint32_t)kFlagAbort};
            }
        }
        __syncthreads();
        const StepWord word = s_word;
        if (word.flags & kFlagAbort) return;
        c = (double)key_float(word.top);
        local = word.step != 0.0;
    }

    const int jfirst = fit ? 0 : L.j0;
    const int jend = fit ? p : L.j1;
    XCol<IPT, XK> xc;
    xc.load(L, ld, jfirst, row0, tg);

    // Wave 0 keeps the bookkeeping (the same in every lane) and takes the step: its
    // inputs are read at the start of the coordinate, and lane 0 writes beta_j and the
    // half-width after the gather, for the next sweep.
    int sweeps = 0, pinned = 0, pinned_last = 0;
    double maxstep = 0.0, last_maxstep = 0.0, objective = 0.0;
    uint32_t stop = 0;

    for (;;) {
        for (int j = jfirst; j < jend; ++j) {
            ++epoch;
            const int jn = (j + 1 < jend) ? j + 1 : jfirst;
            XCol<IPT, XK> xn;
            xn.load(L, ld, jn, row0, tg);
            const bool want_obj = (j == jfirst);
            // the step's per-column inputs: issued here, they arrive during the passes
            const double bj = sbeta[j];
            const double qj = L.q[j], gj = L.gamma[j];
            double trj = trust[j];

            // pass 1: D, N1, N2 of the thread's rows and their fold; the scans to what enters the thread;
            // pass 2: inclusive prefixes at group ends -> per-coordinate sums
            double wv[IPT];
            const bool extra = want_obj || !fit;
            Partial v = partial_identity();
            v.top = (uint32_t)(exp_rows<IPT>(wv, eta, c, s_exptab) + kTopBias);
            if constexpr (EFRON) {
                RV tagg = seg_identity<KV, NC>();
#pragma unroll
                for (int i = 0; i < IPT; ++i) tagg = seg_combine(tagg, row_value<EFRON, XK>(meta[i], wv[i], xc[i]));
                RV exc;
                if constexpr (WAVE) {
                    exc = wave_shift_right(wave_inclusive_scan(tagg));
                } else {
                    RV btot;
                    exc = block_exclusive_scan<KV, NW, NC>(tagg, s_wtot, btot);
                    if (t == 0) publish_aggregate(agg, b, btot, epoch, local);
                    if (!tile_head) {
                        RV carry;
                        if (!look_back<KV, NC>(b, epoch, agg, ctl, s_win, &s_abort, carry)) return;
                        exc = seg_combine(carry, exc);
                    }
                }
                // What pass 2 can form again from the weights and row words is not kept for it: with two waves
                // per SIMD and 8 or 16 rows that spilled (512 x 16, N = 2e6, K = 1e5: 40.2 us per coordinate
                // on dense X and 38.7 on sparse, now 32.0 and 27.7)
                if constexpr (BLOCK * IPT >= 4096) {
#pragma unroll
                    for (int i = 0; i < IPT; ++i) asm volatile("" : "+v"(wv[i]), "+v"(meta[i]));
                }
                if (want_obj) pass2_efron<IPT, XK, true>(v, exc, meta, wv, xc, c);
                else pass2_efron<IPT, XK, false>(v, exc, meta, wv, xc, c);
            } else {
                Vals<NC> loc[KEEP ? IPT : 1], tagg;
                auto row = [&](int i) {
                    Vals<NC> r;
                    r.v[0] = wv[i];
                    r.v[1] = xc[i] * wv[i];
                    if constexpr (NC == 3) r.v[2] = xc[i] * r.v[1];
                    return r;
                };
#pragma unroll
                for (int i = 0; i < IPT; ++i) {
                    tagg = i == 0 ? row(0) : add_kept(tagg, krow[i], row(i));
                    if constexpr (KEEP) loc[i] = tagg;
                }
                Vals<NC> exc;
                if constexpr (WAVE) {
                    exc = dpp_vals<0x138, 0xF>(keep.template wave_scan<NC>(tagg));
                } else {
                    Vals<NC> btot;
                    exc = keep.template block_scan<NC>(tagg, s_vtot, btot);
                    if (t == 0) {
                        RV a;
                        a.f = keep.tile_flag;
#pragma unroll
                        for (int k = 0; k < NC; ++k) a.v[k] = btot.v[k];
                        publish_aggregate(agg, b, a, epoch, local);
                    }
                    if (!tile_head) {
                        RV carry;
                        if (!look_back<KV, NC>(b, epoch, agg, ctl, s_win, &s_abort, carry)) return;
#pragma unroll
                        for (int k = 0; k < NC; ++k) exc.v[k] = fma(carry.v[k], keep.carry, exc.v[k]);
                    }
                }
                Vals<NC> run = exc;
                auto prefix = [&](int i, double (&out)[NC]) {
                    if constexpr (KEEP) {
#pragma unroll
                        for (int k = 0; k < NC; ++k) out[k] = fma(exc.v[k], kall[i], loc[KEEP ? i : 0].v[k]);
                    } else {
                        run = add_kept(run, krow[i], row(i));   // called in row order
#pragma unroll
                        for (int k = 0; k < NC; ++k) out[k] = run.v[k];
                    }
                };
                if (want_obj) pass2_breslow<IPT, NC, true>(v, meta, c, prefix);
                else pass2_breslow<IPT, NC, false>(v, meta, c, prefix);
            }
            if (want_obj) {
#pragma unroll
                for (int i = 0; i < IPT; ++i) v.obj -= (meta[i] & kEventBit) ? eta[i] : 0.0;
                v = block_reduce_partial<NW, true>(v, s_red);
            } else {
                v = block_reduce_partial<NW, false>(v, s_red);
            }

            // wave 0 publishes, gathers every workgroup's record and takes the step; the others wait for it
            if (w == 0) {
                if (lane == NW - 1) publish_partial(part, G, b, v, epoch, extra, local);
                Partial tot;
                StepWord word = {0.0, 0u, kFlagAbort};
                if (gather_wave<!WAVE>(part, G, epoch, extra, ctl, tot)) {
                    uint32_t flags = tot.err ? kFlagNumeric : 0u;
                    const double g1 = -qj + tot.c1, g2 = tot.c2, m2 = tot.m2;
                    double step = 0.0;
                    if (fit && !tot.err) {
                        int pin = 0;
                        step = ccd_step(bj, g1, g2, m2, gj, &trj, &pin);
                        maxstep = fmax(maxstep, fabs(step));
                        pinned += pin;
                        if (j == jend - 1) {
                            ++sweeps;
                            double bmax = 1.0;
                            for (int k = lane; k < p; k += kWave) bmax = fmax(bmax, fabs(k == j ? bj + step : sbeta[k]));
#pragma unroll
                            for (int o = kWave / 2; o >= 1; o >>= 1) bmax = fmax(bmax, __shfl_xor(bmax, o, kWave));
                            if (maxstep <= L.tol * bmax) flags |= kFlagConverged;
                            else if (sweeps >= L.max_sweeps) flags |= kFlagSweepLimit;
                            last_maxstep = maxstep;
                            pinned_last = pinned;
                            maxstep = 0.0;
                            pinned = 0;
                        }
                        if (lane == 0) {
                            trust[j] = trj;
                            sbeta[j] = bj + step;
                        }
                    }
                    word = StepWord{step, tot.top, flags};
                    if (lane == 0) s_word = word;
                    if (writer) {
                        L.g1[j] = g1;
                        L.g2[j] = g2;
                        L.m2[j] = m2;
                    }
                    if (want_obj) {
                        objective = tot.obj;
                        if (fit) {
                            // the penalty at the sweep's start (beta_j is already replaced)
                            double pen = 0.0;
                            for (int k = lane; k < p; k += kWave) pen = fma(L.gamma[k], fabs(k == j ? bj : sbeta[k]), pen);
#pragma unroll
                            for (int o = kWave / 2; o >= 1; o >>= 1) pen += __shfl_xor(pen, o, kWave);
                            objective += pen;
                        }
                    }
                } else if (lane == 0) {
                    s_word = word;
                }
            }
            __syncthreads();
            const StepWord word = s_word;
            if (word.flags & (kFlagAbort | kFlagNumeric)) {
                if (word.flags & kFlagAbort) return;
                stop = kFlagNumeric;
                break;
            }
            const double step = word.step;
            c = fma((double)((int)word.top - kTopBias), kTopStep, c);
            if (step != 0.0) {
#pragma unroll
                for (int i = 0; i < IPT; ++i) eta[i] = fma(xc[i], step, eta[i]);
            }
            xc = xn;
            if (word.flags & (kFlagConverged | kFlagSweepLimit)) {
                stop = word.flags;
                break;
            }
        }
        if (stop || !fit) break;
    }

    if (b == 0) {
        // wave 0 holds the bookkeeping; beta is in LDS (written before the last barrier), the
        // derivatives were written by this workgroup's thread 0
        auto seen = [](const double *v) { return __hip_atomic_load(v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
        __threadfence();
        __syncthreads();
        for (int j = t; j < p; j += BLOCK) {
            L.hout[j] = sbeta[j];
            L.hout[p + j] = seen(L.g1 + j);
            L.hout[2 * p + j] = seen(L.g2 + j);
            L.hout[3 * p + j] = seen(L.m2 + j);
        }
        if (t == 0) {
            double *result = L.hout + 4 * (int64_t)p;
            result[kResSweeps] = sweeps;
            result[kResLastStep] = last_maxstep;
            result[kResObjective] = objective;
            result[kResPinned] = pinned_last;
            result[kResConverged] = (stop & kFlagConverged) ? 1.0 : 0.0;
            result[kResNumeric] = (stop & kFlagNumeric) ? 1.0 : 0.0;
            result[kResAborted] = abort_raised(ctl) ? 1.0 : 0.0;
            result[kResCompleted] = 1.0;
        }
    }
}

// Before the persistent kernel: the synchronisation words cleared, the start point read from
// host memory once (not by every workgroup).
__global__ __launch_bounds__(256) void ccd_prepare_kernel(uint32_t *words, int64_t nwords, const double *beta0,
                                                          double *beta, int p)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < nwords) words[i] = 0u;
    if (i < p) beta[i] = beta0 ? beta0[i] : 0.0;
}

// ------------------------------------------------------------------ raw segmented scan

constexpr int kScanBlock = 1024;

// Where one scan's workgroups meet.  The scan is an ordinary launch: a workgroup takes the next
// tile by a ticket, so every tile it waits for belongs to a workgroup that has already started
// (and publishes its aggregate before it waits itself).  Tickets and epochs go on from call to
// call on the same words, so nothing is cleared between.
struct ScanSync {
    SyncCtl *ctl;            // abort; pad[0]: the ticket counter
    Packet *agg;             // one packet per tile
    uint32_t epoch, ticket0; // of this call
    uint32_t *host_abort;    // set when a wait has timed out (may be NULL)
};

// VEC: a and out are 16-byte aligned and head is IPT-byte aligned, so that a whole tile's rows move
// 16 bytes per access (8-byte accesses IPT * 8 bytes apart touch every line IPT times).
template <int IPT, bool VEC>
__global__ __launch_bounds__(kScanBlock) void segscan_kernel(const double *a, const uint8_t *head, double *out,
                                                             int64_t n, ScanSync S)
{
    const PacketArray agg = packet_array(S.agg, sizeof(Packet) * gridDim.x);
    constexpr int NW = kScanBlock / kWave;
    __shared__ SegVal<1> s_wtot[NW];
    __shared__ SegVal<1> s_win[kMaxGroups / kWave];
    __shared__ int s_abort, s_tile;
    const int t = threadIdx.x;
    if (t == 0) {
        s_abort = 0;
        s_tile = (int)(__hip_atomic_fetch_add(&S.ctl->pad[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - S.ticket0);
    }
    __syncthreads();
    const int b = __builtin_amdgcn_readfirstlane(s_tile);
    const int64_t tile0 = (int64_t)b * kScanBlock * IPT;
    const int64_t row0 = tile0 + (int64_t)t * IPT;
    const bool whole = VEC && tile0 + kScanBlock * IPT <= n;
    SegVal<1> e[IPT];
    SegVal<1> tagg = seg_identity<1>();
    if (whole) {
        double v[IPT];
        load_rows<IPT>(v, a + row0);
        uint32_t h[IPT];
        if constexpr (IPT == 16) {
            const uint4 w = *reinterpret_cast<const uint4 *>(head + row0);
            const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int i = 0; i < IPT; ++i) h[i] = (ws[i / 4] >> (8 * (i % 4))) & 0xffu;
        } else if constexpr (IPT == 8) {
            const uint2 w = *reinterpret_cast<const uint2 *>(head + row0);
#pragma unroll
            for (int i = 0; i < IPT; ++i) h[i] = ((i < 4 ? w.x : w.y) >> (8 * (i % 4))) & 0xffu;
        } else if constexpr (IPT == 4) {
            const uint32_t w = *reinterpret_cast<const uint32_t *>(head + row0);
#pragma unroll
            for (int i = 0; i < IPT; ++i) h[i] = (w >> (8 * i)) & 0xffu;
        } else {
#pragma unroll
            for (int i = 0; i < IPT; ++i) h[i] = head[row0 + i];
        }
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            e[i].f = (row0 + i == 0 || h[i] != 0) ? 1u : 0u;
            e[i].v[0] = v[i];
            tagg = seg_combine(tagg, e[i]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            const int64_t r = row0 + i;
            if (r < n) {
                e[i].f = (r == 0 || head[r] != 0) ? 1u : 0u;
                e[i].v[0] = a[r];
            } else {
                e[i].f = 1u;
                e[i].v[0] = 0.0;
            }
            tagg = seg_combine(tagg, e[i]);
        }
    }
    SegVal<1> btot;
    SegVal<1> exc = block_exclusive_scan<1, NW>(tagg, s_wtot, btot);
    if (t == 0) publish_aggregate<1>(agg, b, btot, S.epoch, false);
    const bool tile_head = tile0 >= n || tile0 == 0 || head[tile0] != 0;
    if (!tile_head) {
        SegVal<1> carry;
        if (!look_back<1>(b, S.epoch, agg, S.ctl, s_win, &s_abort, carry)) {
            if (t == 0 && S.host_abort) __hip_atomic_store(S.host_abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            return;
        }
        exc = seg_combine(carry, exc);
    }
    SegVal<1> run = exc;
    if (whole && IPT % 2 == 0) {
        double o[IPT];
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            run = seg_combine(run, e[i]);
            o[i] = run.v[0];
        }
#pragma unroll
        for (int i = 0; i + 1 < IPT; i += 2) *reinterpret_cast<double2 *>(out + row0 + i) = double2{o[i], o[i + 1]};
    } else {
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            run = seg_combine(run, e[i]);
            if (row0 + i < n) out[row0 + i] = run.v[0];
        }
    }
}

// ------------------------------------------------------------------ host launchers

namespace {

// Dynamic LDS of one persistent workgroup: beta.
size_t ccd_smem_bytes(int, int p)
{
    return sizeof(double) * (size_t)p;
}

// One instantiation per workgroup shape (kShapes; some are for Efron's ties alone).
template <int XK, bool EFRON, bool WAVE>
const void *ccd_fn(int threads, int ipt)
{
    if (threads == 512) {
        if constexpr (EFRON) {
            if (ipt == 1) return reinterpret_cast<const void *>(&ccd_kernel<512, 1, XK, EFRON, WAVE>);
            if (ipt == 2) return reinterpret_cast<const void *>(&ccd_kernel<512, 2, XK, EFRON, WAVE>);
            if (ipt == 4) return reinterpret_cast<const void *>(&ccd_kernel<512, 4, XK, EFRON, WAVE>);
        }
        if (ipt == 8) return reinterpret_cast<const void *>(&ccd_kernel<512, 8, XK, EFRON, WAVE>);
        if (ipt == 16) return reinterpret_cast<const void *>(&ccd_kernel<512, 16, XK, EFRON, WAVE>);
    } else if (threads == 256) {
        if (ipt == 1) return reinterpret_cast<const void *>(&ccd_kernel<256, 1, XK, EFRON, WAVE>);
        if (ipt == 2) return reinterpret_cast<const void *>(&ccd_kernel<256, 2, XK, EFRON, WAVE>);
        if (ipt == 4) return reinterpret_cast<const void *>(&ccd_kernel<256, 4, XK, EFRON, WAVE>);
        if (ipt == 8) return reinterpret_cast<const void *>(&ccd_kernel<256, 8, XK, EFRON, WAVE>);
    }
    return nullptr;
}

template <bool WAVE>
const void *ccd_function_w(int threads, int ipt, int xk, bool efron)
{
    if (xk == 2) return efron ? ccd_fn<2, true, WAVE>(threads, ipt) : ccd_fn<2, false, WAVE>(threads, ipt);
    if (xk == 1) return efron ? ccd_fn<1, true, WAVE>(threads, ipt) : ccd_fn<1, false, WAVE>(threads, ipt);
    return efron ? ccd_fn<0, true, WAVE>(threads, ipt) : ccd_fn<0, false, WAVE>(threads, ipt);
}

// xk: 0 dense X, 1 indicator X, 2 sparse values (see XCol)
const void *ccd_function(int threads, int ipt, int xk, bool efron, bool wave)
{
    return wave ? ccd_function_w<true>(threads, ipt, xk, efron) : ccd_function_w<false>(threads, ipt, xk, efron);
}

// Workgroups of the persistent kernel that fit on one compute unit; every variant of the shape
// (indicator or sparse X, Efron, wave-aligned layout) must fit, since a handle may run any of them.
int occupancy_for(int threads, int ipt, int p, int *blocks)
{
    *blocks = 1 << 30;
    if (!ccd_function(threads, ipt, 0, true, false)) return (int)hipErrorInvalidValue;
    for (int v = 0; v < 12; ++v) {
        const void *fn = ccd_function(threads, ipt, v % 3, ((v / 3) & 1) != 0, ((v / 3) & 2) != 0);
        if (!fn) continue;
        int nb = 0;
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, threads, ccd_smem_bytes(ipt, p));
        if (e != hipSuccess) return (int)e;
        *blocks = nb < *blocks ? nb : *blocks;
    }
    return (int)hipSuccess;
}

int device_cus(int *cus)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    return (int)hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev);
}

}  // namespace

int max_resident_groups(int threads, int ipt, int p, int *groups, std::string &err)
{
    *groups = 0;
    int cus = 0;
    if (device_cus(&cus) != (int)hipSuccess || cus <= 0) {
        err = "cannot query the device's compute-unit count";
        return -3;
    }
    // Twelve occupancy queries take tens of microseconds, as long as a small refit's kernels: asked
    // once per device and shape at the most columns (the most LDS); a smaller p then fits too.
    static std::mutex mu;
    static std::map<std::array<int, 3>, int> at_most_columns;
    int dev = -1, blocks = 0;
    (void)hipGetDevice(&dev);
    {
        std::lock_guard<std::mutex> lock(mu);
        const auto key = std::array<int, 3>{dev, threads, ipt};
        const auto it = at_most_columns.find(key);
        if (it != at_most_columns.end()) {
            blocks = it->second;
        } else {
            if (occupancy_for(threads, ipt, (int)kMaxCcdP, &blocks) != (int)hipSuccess) {
                err = "occupancy query failed";
                return -3;
            }
            at_most_columns[key] = blocks;
        }
    }
    if (blocks < 1 && occupancy_for(threads, ipt, p, &blocks) != (int)hipSuccess) {
        err = "occupancy query failed";
        return -3;
    }
    *groups = blocks >= 1 ? (cus < kMaxGroups ? cus : kMaxGroups) : 0;   // one workgroup per compute unit
    return 0;
}

int launch_ccd(const LaunchShape &shape, const CcdLaunch &L, hipStream_t stream, hipEvent_t ev0,
               hipEvent_t ev1)
{
    const int64_t words = (int64_t)(sync_scratch_bytes(shape.grid) / sizeof(uint32_t));
    const int64_t most = words > L.p ? words : L.p;
    ccd_prepare_kernel<<<(unsigned)((most + 255) / 256), 256, 0, stream>>>(static_cast<uint32_t *>(L.ctl), words, L.beta0,
                                                                          L.beta, L.p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
    if (ev0 && (e = hipEventRecord(ev0, stream)) != hipSuccess) return (int)e;
    CcdLaunch arg = L;
    arg.spread = shape.spread;
    void *args[] = {&arg};
    const size_t smem = ccd_smem_bytes(shape.ipt, L.p);
    const void *fn = ccd_function(shape.threads, shape.ipt, L.xvals ? 2 : (L.xbits ? 1 : 0), L.efron != 0, shape.wave);
    if (!fn) return (int)hipErrorInvalidValue;
    e = hipLaunchCooperativeKernel(fn, dim3(shape.grid * shape.spread), dim3(shape.threads), args, (unsigned)smem, stream);
    if (e != hipSuccess) return (int)e;
    if (ev1 && (e = hipEventRecord(ev1, stream)) != hipSuccess) return (int)e;
    return (int)hipSuccess;
}

namespace {

constexpr size_t kScanScratchBytes = 256 + sizeof(Packet) * kMaxGroups;
static_assert(sizeof(SyncCtl) <= 256, "control block");

// Rows per thread and workgroups for n rows; 0 rows: too long for one workgroup per compute unit.
int scan_shape(int64_t n, int cus, int64_t *grid)
{
    for (int c : {1, 2, 4, 8, 16}) {
        *grid = (n + (int64_t)kScanBlock * c - 1) / ((int64_t)kScanBlock * c);
        if (*grid <= cus && *grid <= kMaxGroups) return c;
    }
    return 0;
}

template <int IPT>
void launch_segscan_ipt(unsigned grid, const double *a, const uint8_t *head, double *b, int64_t n, const ScanSync &S,
                        hipStream_t stream)
{
    const bool vec = (reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) % 16 == 0 &&
                     reinterpret_cast<uintptr_t>(head) % IPT == 0;
    if (vec) segscan_kernel<IPT, true><<<grid, kScanBlock, 0, stream>>>(a, head, b, n, S);
    else segscan_kernel<IPT, false><<<grid, kScanBlock, 0, stream>>>(a, head, b, n, S);
}

hipError_t launch_segscan(int ipt, unsigned grid, const double *a, const uint8_t *head, double *b, int64_t n,
                          const ScanSync &S, hipStream_t stream)
{
    switch (ipt) {
    case 1: launch_segscan_ipt<1>(grid, a, head, b, n, S, stream); break;
    case 2: launch_segscan_ipt<2>(grid, a, head, b, n, S, stream); break;
    case 4: launch_segscan_ipt<4>(grid, a, head, b, n, S, stream); break;
    case 8: launch_segscan_ipt<8>(grid, a, head, b, n, S, stream); break;
    default: launch_segscan_ipt<16>(grid, a, head, b, n, S, stream); break;
    }
    return hipGetLastError();
}

ScanSync scan_sync(void *base, uint32_t epoch, uint32_t ticket0, uint32_t *host_abort)
{
    char *cb = static_cast<char *>(base);
    return ScanSync{reinterpret_cast<SyncCtl *>(cb), reinterpret_cast<Packet *>(cb + 256), epoch, ticket0, host_abort};
}

constexpr int kMaxDevices = 64;

}  // namespace

// ------------------------------------------------------------------ scan slots
//
// The synchronisation words of cox_segscan_f64: kScanSlots sets in the library's device memory
// (139 KB per GPU), one held by each call while it runs, so calls on several threads and streams
// do not meet.  A call that finds all of them taken allocates its own.  With an allocation, a clear,
// a cooperative launch, a copy of the abort word and a release on every call a scan of 1e6 rows
// took 61 us, now 20, most of it the launch and the wait for it.
constexpr int kScanSlots = 32;
static __device__ __align__(256) unsigned char scan_slots[kScanSlots * kScanScratchBytes];

namespace {

struct ScanSlot {
    bool taken = false, broken = false;   // broken: a wait timed out or the device failed; not used again
    uint32_t epoch = 0, ticket = 0;       // of the last call; the ticket counter's value
};

struct ScanSlots {
    std::mutex mu;
    void *base[kMaxDevices] = {};
    ScanSlot slot[kMaxDevices][kScanSlots];
    uint32_t *aborts = nullptr;           // pinned, one word per device and slot
};

ScanSlots &scan_slot_table()
{
    static ScanSlots *t = new ScanSlots;
    return *t;
}

// A free slot of the current device, or -1.
int take_scan_slot(int dev, void **base, uint32_t **host_abort)
{
    ScanSlots &T = scan_slot_table();
    std::lock_guard<std::mutex> lock(T.mu);
    if (!T.aborts) {
        void *p = nullptr;
        const size_t bytes = sizeof(uint32_t) * kMaxDevices * kScanSlots;
        if (hipHostMalloc(&p, bytes, hipHostMallocPortable) != hipSuccess) {
            (void)hipGetLastError();
            return -1;
        }
        T.aborts = static_cast<uint32_t *>(p);
        for (int i = 0; i < kMaxDevices * kScanSlots; ++i) T.aborts[i] = 0u;
    }
    if (!T.base[dev] &&
        (hipGetSymbolAddress(&T.base[dev], HIP_SYMBOL(scan_slots)) != hipSuccess || !T.base[dev])) {
        (void)hipGetLastError();
        T.base[dev] = nullptr;
        return -1;
    }
    for (int k = 0; k < kScanSlots; ++k) {
        ScanSlot &s = T.slot[dev][k];
        if (s.taken || s.broken) continue;
        s.taken = true;
        if (++s.epoch == 0u) ++s.epoch;   // packets start out with epoch 0
        *base = static_cast<char *>(T.base[dev]) + (size_t)k * kScanScratchBytes;
        *host_abort = T.aborts + dev * kScanSlots + k;
        return k;
    }
    return -1;
}

void release_scan_slot(int dev, int k, bool ok)
{
    ScanSlots &T = scan_slot_table();
    std::lock_guard<std::mutex> lock(T.mu);
    T.slot[dev][k].broken = !ok;
    T.slot[dev][k].taken = false;
}

}  // namespace

int segscan_f64(const double *a, const uint8_t *head, double *b, int64_t n, hipStream_t stream)
{
    if (n < 0 || (n > 0 && (!a || !head || !b))) return -1;
    if (n == 0) return 0;
    int cus = 0, dev = -1;
    if (device_cus(&cus) != (int)hipSuccess || cus <= 0 || hipGetDevice(&dev) != hipSuccess) return -3;
    int64_t grid = 0;
    const int ipt = scan_shape(n, cus, &grid);
    if (!ipt) return -5;
    void *base = nullptr;
    uint32_t *host_abort = nullptr;
    // (a stream that is being captured cannot wait for its result: that call is refused further down)
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    const bool plain = hipStreamIsCapturing(stream, &capture) == hipSuccess && capture == hipStreamCaptureStatusNone;
    if (!plain) (void)hipGetLastError();
    const int k = plain && dev >= 0 && dev < kMaxDevices ? take_scan_slot(dev, &base, &host_abort) : -1;
    if (k >= 0) {
        ScanSlot &slot = scan_slot_table().slot[dev][k];   // ours until released
        hipError_t e = launch_segscan(ipt, (unsigned)grid, a, head, b, n,
                                      scan_sync(base, slot.epoch, slot.ticket, host_abort), stream);
        if (e == hipSuccess) {
            slot.ticket += (uint32_t)grid;
            e = hipStreamSynchronize(stream);
        }
        const bool ok = e == hipSuccess && __atomic_load_n(host_abort, __ATOMIC_ACQUIRE) == 0u;
        release_scan_slot(dev, k, ok);
        return ok ? 0 : -3;
    }
    void *scratch = nullptr;
    if (device_malloc(&scratch, kScanScratchBytes) != hipSuccess) return -2;
    const ScanSync S = scan_sync(scratch, 1u, 0u, nullptr);
    uint32_t aborted = 0;
    hipError_t e = hipMemsetAsync(scratch, 0, kScanScratchBytes, stream);
    if (e == hipSuccess) e = launch_segscan(ipt, (unsigned)grid, a, head, b, n, S, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e == hipSuccess) e = hipMemcpy(&aborted, &S.ctl->abort, sizeof(uint32_t), hipMemcpyDeviceToHost);
    (void)hipFree(scratch);
    return (e != hipSuccess || aborted) ? -3 : 0;
}

// ------------------------------------------------------------------ the scan without allocation

// Synchronisation words of segscan_f64_noalloc: the control block and one aggregate
// packet per workgroup (at most kMaxGroups), in library-owned device memory that
// exists once per GPU for the life of the process.  Host code never uses this name
// as an address: its per-device address comes from hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[kScanScratchBytes];

namespace {

std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// The device address of `scratch` on the current device, looked up once per device.
int scratch_address(void **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return -3;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return -3;
        }
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return 0;
}

// Zero `words` 32-bit words (a fill kernel rather than a memset node, so the call can
// sit in captured work).
__global__ __launch_bounds__(256) void zero_words_kernel(uint32_t *p, int words)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < words) p[i] = 0u;
}

}  // namespace

int segscan_f64_noalloc(const double *a, const uint8_t *head, double *b, int64_t n, hipStream_t stream)
{
    if (n < 0 || (n > 0 && (!a || !head || !b))) return -1;
    if (n == 0) return 0;
    int cus = 0;
    if (device_cus(&cus) != (int)hipSuccess || cus <= 0) return -3;
    int64_t grid = 0;
    const int ipt = scan_shape(n, cus, &grid);
    if (!ipt) return -5;
    void *base = nullptr;
    if (scratch_address(&base) != 0) return -3;
    const ScanSync S = scan_sync(base, 1u, 0u, nullptr);
    // the previous call's packets carry the same epoch: clear them before this scan reads any
    const int words = (int)((256 + sizeof(Packet) * (size_t)grid) / sizeof(uint32_t));
    hipLaunchKernelGGL(zero_words_kernel, dim3((words + 255) / 256), dim3(256), 0, stream,
                       reinterpret_cast<uint32_t *>(base), words);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = launch_segscan(ipt, (unsigned)grid, a, head, b, n, S, stream);
    uint32_t aborted = 0;
    if (e == hipSuccess)
        e = hipMemcpyAsync(&aborted, &S.ctl->abort, sizeof(uint32_t), hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    return (e != hipSuccess || aborted) ? -3 : 0;
}

}  // namespace coxmi
