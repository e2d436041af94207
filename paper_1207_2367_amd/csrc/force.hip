// Evaluation step of the Hermite scheme on gfx950: acceleration, jerk, snap
// and potential of the active particles against all sources of their
// cluster (paper Sect. 3, item 2, with the softened potential of Sect. 2),
// plus the split-source reduction (the paper's "Bfactor", Sect. 3).
//
// Design (CDNA4, wave64):
//   - one workgroup = NW waves; each wave holds GI = 64 / LPI active
//     particles, LPI lanes per particle; the i-particle lives in registers;
//   - sources are staged through LDS in tiles of NT = 64 NW records (one
//     16-byte aligned record per source), loaded coalesced from the
//     structure-of-arrays source arrays by the whole workgroup; lane slot js
//     of an i-particle takes tile entries js, js + LPI, ...; with LPI = 1
//     every LDS read is a broadcast;
//   - the pair loop is pure vector ALU: no matrix cores, the work is not a
//     dense contraction (every pair needs a reciprocal square root and
//     nonlinear terms);
//   - mixed precision: r_j - r_i, r^2 and 1/r (v_rsq_f32 seed + one FP64
//     Newton step) in FP64, and with them the acceleration, jerk (from FP64
//     velocity differences) and potential terms, summed in FP64; the snap
//     term in FP32 from the rounded r_j - r_i, jerk vector and coefficients
//     and the FP32 acceleration differences, summed over at most 64 pairs
//     per lane in FP32 and folded into double-single (hi, lo) accumulators
//     by an error-free two-sum.  Per-term FP32 rounding in a sum with
//     cancellation grows with the sum's condition number, so the quantities
//     held to 1e-6 per particle (acceleration, jerk, potential) stay FP64;
//     the snap is the least amplified: the fifth-derivative estimate of the
//     step criterion multiplies the acceleration's absolute error by
//     ~720/h^5 but the snap's by at most ~1/h^3;
//   - the LPI lanes of a particle are combined by cross-lane register moves in
//     a fixed order (lane_sum, LaneSums);
//   - the FP64 passes take 1/r from the same FP32 seed, refined to FP64
//     accuracy by one third-order step;
//   - the potential energy (energy_kernel) takes every pair once, with a
//     cyclic half-window per particle that gives every workgroup equal work;
//   - grid.y = B splits the sources (whole units, sizes alike; a cluster with
//     fewer units uses fewer splits, the rest exit at once); partial results
//     go to a [B][10][n_act] buffer that a second kernel sums in fixed order
//     b = 0 .. B_c-1 (reduce_split here, the corrector's kernel in a block
//     step, or the correction phase of the device-resident loop), so the
//     result does not depend on scheduling (no float atomics anywhere);
//   - the per-workgroup body (force_block) lives in force_body.h, shared by
//     the launch kernel here and the device-resident block-step loop;
//   - a block step's evaluation skips the potential (template flag PHI).
#include <cmath>

#include "force_body.h"

namespace nb {

namespace {

// One source of the energy pass in LDS.
struct alignas(16) PotSrc {
    double x, y, z, m;
};

// Softening of the energy pass: none; one whose square is a normal FP32 number,
// which rinv_f64 needs; one whose square is not.  With the last, the particle's
// own slot (r2 = eps2, masked) has no finite 1/r, so masked slots are put at
// r2 = 1: two more instructions per pair of a masked tile, 0.6-1 % of the pass.
enum : int { EPS_NONE, EPS_NORMAL, EPS_ODD };

// Potential terms of one LDS tile of NT sources for the IPT particles of one
// lane: phi -= m_j / r_ij, FP64.  MASK keeps only the tile slots lo <= t <= hi
// of each particle.
template <int NT, int IPT, bool MASK, int EPS>
__device__ __forceinline__ void pot_tile(const PotSrc *s, const double *xi, const double *yi,
                                         const double *zi, double eps2, const int *lo,
                                         const int *hi, double *phi)
{
#pragma unroll 4
    for (int t = 0; t < NT; ++t) {
        const double sx = s[t].x, sy = s[t].y, sz = s[t].z, sm = s[t].m;
#pragma unroll
        for (int u = 0; u < IPT; ++u) {
            const double dx = sx - xi[u], dy = sy - yi[u], dz = sz - zi[u];
            double r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2)));
            if constexpr (MASK && EPS == EPS_ODD)
                r2 = (t >= lo[u] && t <= hi[u]) ? r2 : 1.0;
            double rinv = rinv_f64(r2);
            if constexpr (EPS == EPS_NONE)
                rinv = r2 > 0.0 ? rinv : 0.0;
            // the mass is masked, not 1/r: the compiler would branch around 1/r
            double m = sm;
            if constexpr (MASK)
                m = (t >= lo[u] && t <= hi[u]) ? m : 0.0;
            phi[u] = fma(-m, rinv, phi[u]);
        }
    }
}

// Which (i-block, split) a workgroup of a launch takes.  The hardware deals
// consecutive workgroups (x fastest) to the NXCD XCDs in turn, and each XCD
// has an L2 of its own: taken as (blockIdx.x, blockIdx.y), the i-blocks that
// run side by side on one XCD belong to several splits, and every XCD
// fetches every split's source records from memory.  Renumbered so that XCD
// k takes the k-th contiguous run of the pairs in x-fastest order, the
// workgroups resident on one XCD walk the same split's tiles together and
// share them in its L2.  A bijection of the grid for any size: the first
// (total mod NXCD) XCDs get one pair more.
__device__ __forceinline__ void xcd_order(int64_t &g, int &b)
{
    constexpr uint64_t NXCD = 8;
    const uint64_t nx = gridDim.x, tot = nx * gridDim.y;
    const uint64_t id = blockIdx.x + (uint64_t)blockIdx.y * nx;
    const uint64_t x = id % NXCD, r = id / NXCD, q = tot / NXCD, rem = tot % NXCD;
    const uint64_t l = x < rem ? x * (q + 1) + r : rem * (q + 1) + (x - rem) * q + r;
    g = (int64_t)(l % nx);
    b = (int)(l / nx);
}

// PHI: also sum the potential (nbody_force, the start-up pass); a block
// step's evaluation does not need it (the energy has its own pass).  IPT:
// active particles per lane group.
// Waves per SIMD that the registers are allotted for: as many as a shape
// holds with hardly a spill outside its pair loop (left alone, the compiler
// spends registers on deeper unrolling and drops to two waves).  FP32-pair with
// one particle per lane group, 65,536 sources: 1000 active 109.1 us with three
// and 103.1 with four.
constexpr int force_waves(int prec, int lpi, int ipt)
{
    if (ipt == 2)
        return prec == PREC_PAIR32 && lpi == 1 ? 2 : 3;
    return 4;
}

// Whether a tile's sources are fetched one tile ahead (force_block).  Not by
// one lane per particle with FP32 pairs: those tiles are 256 short pairs per
// lane, four waves hide the fetch, and its registers are missed in the pair
// loop (65,536 active, 524,288 sources: 37.3 ms with, 36.9 without).
constexpr bool force_ahead(int prec, int lpi)
{
    return !(prec == PREC_PAIR32 && lpi == 1);
}

// Sources of an evaluation: with the potential (nbody_force, at the stored
// state's own times) the FP64 state or the caller's arrays as they stand, so
// that no packing pass runs first; in a block step the predicted records.
template <int PREC, bool PHI>
using SrcOf = typename std::conditional<PHI, JSrc, typename Smem<PREC>::R>::type;

template <int PREC, int LPI, int NW, bool EPS0, bool PHI, int IPT>
__global__ __launch_bounds__(NW * 64, force_waves(PREC, LPI, IPT)) void force_kernel(
    SrcOf<PREC, PHI> J, ForceWork w, ForceOut out, double *part,
    int64_t n_act_total, double eps2)
{
    int64_t g;
    int b;
    xcd_order(g, b);
    force_block<PREC, LPI, NW, EPS0, PHI, IPT, force_ahead(PREC, LPI)>(J, w, out, part, n_act_total, eps2, g, b);
}

// Potential energy of the stored state (paper Sect. 5.1): every unordered
// pair of a cluster once, FP64.  Particle i (local index l in a cluster of
// size n_c) takes the sources l + 1 .. l + W_l taken cyclically, with
// W_l = (n_c - 1) / 2 for odd n_c and, for even n_c, n_c / 2 for l < n_c / 2
// and n_c / 2 - 1 otherwise: each pair at cyclic distance d < n_c / 2 is
// then taken by exactly one of its ends, and the pair at d = n_c / 2 by the
// end with the smaller index, so sum_l W_l = n_c (n_c - 1) / 2 and every
// workgroup does the same work (no triangle).  A workgroup holds IB = 256 IPT
// consecutive particles, IPT per lane (each source read from LDS serves IPT
// pairs: with one, the two 128-bit reads per pair take 64 of the 71 cycles of
// its vector instructions; 100,003 bodies 2.38 and 2.28 ms with 1 and 2); the
// union of their windows (virtual positions ib0 + 1 .. last + W, folded back
// into the cluster) goes through LDS in tiles of 256, split over grid.y = B;
// lanes mask only the tiles at the two ends of the union.  Output: partial
// sums -sum m_j / r_ij per particle and split, out[b n + i].  Nothing is done
// if the error word says that the particles are not at one time.
template <int EPS, int IPT>
__global__ __launch_bounds__(256) void energy_kernel(const double *X, const double *Y,
                                                     const double *Z, const double *M,
                                                     ForceWork w, double *out, int64_t n,
                                                     double eps2)
{
    constexpr int NT = 256, IB = NT * IPT;
    __shared__ PotSrc s[NT];
    if (*w.err & ERR_STATE)
        return;
    const int64_t g = blockIdx.x;
    const int b = blockIdx.y;
    int64_t gfirst = 0, o0 = 0, nc = n;
    if (w.blk_cluster) {
        const int c = w.blk_cluster[g];
        if (c < 0)
            return;  // grid padding past the last i-block
        gfirst = w.blk_first[c];
        o0 = w.off[c];
        nc = w.off[c + 1] - o0;
    }
    const int64_t ib0 = (g - gfirst) * IB;          // local index of lane 0's first particle
    const int64_t last = (ib0 + IB < nc ? ib0 + IB : nc) - 1;
    const int tid = threadIdx.x;
    const int64_t half = nc / 2;
    const int64_t wmin = (nc & 1) ? half : half - 1;   // smallest window of the cluster
    int64_t l[IPT], wl[IPT];
    double xi[IPT], yi[IPT], zi[IPT], phi[IPT];
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
        l[u] = ib0 + tid + u * NT;
        wl[u] = (nc & 1) ? half : (l[u] < half ? half : half - 1);
        const int64_t i = o0 + (l[u] < nc ? l[u] : ib0);
        xi[u] = X[i];
        yi[u] = Y[i];
        zi[u] = Z[i];
        phi[u] = 0.0;
    }

    // this split's share of the union of the windows, in whole tiles
    const int64_t u_beg = ib0 + 1, len = last + half + 1 - u_beg;
    const int64_t used = splits_used(len, w.split, NT);
    const int64_t u0 = u_beg + (b < used ? split_begin(len, used, NT, b) : len);
    const int64_t u1 = u_beg + (b < used ? split_begin(len, used, NT, b + 1) : len);

    for (int64_t t0 = u0; t0 < u1; t0 += NT) {
        __syncthreads();
        const int64_t v = t0 + tid;
        if (v < u1) {
            const int64_t j = o0 + (v < nc ? v : v - nc);   // v < 2 n_c always
            s[tid] = PotSrc{X[j], Y[j], Z[j], M[j]};
        } else {
            s[tid] = PotSrc{NULL_POS, NULL_POS, NULL_POS, 0.0};
        }
        __syncthreads();
        // slots t of this tile with 1 <= t0 + t - l <= w_l; every particle's
        // range covers the whole tile when t0 > last and t0 + NT - 1 <= ib0 + wmin
        int lo[IPT], hi[IPT];
        if (t0 > last && t0 + NT - 1 <= ib0 + wmin) {
            pot_tile<NT, IPT, false, EPS>(s, xi, yi, zi, eps2, lo, hi, phi);
        } else {
#pragma unroll
            for (int u = 0; u < IPT; ++u) {
                const int64_t a = l[u] + 1 - t0, z = l[u] + wl[u] - t0;
                lo[u] = a < 0 ? 0 : (a > NT ? NT : (int)a);
                hi[u] = z < -1 ? -1 : (z > NT - 1 ? NT - 1 : (int)z);
            }
            pot_tile<NT, IPT, true, EPS>(s, xi, yi, zi, eps2, lo, hi, phi);
        }
    }
#pragma unroll
    for (int u = 0; u < IPT; ++u)
        if (l[u] < nc)
            out[(int64_t)b * n + o0 + l[u]] = phi[u];
}

// Sum the B split-source partials of every active slot (Table 1, section 4
// of the paper) in a fixed order: R lanes per (quantity, active slot), lane r
// summing the splits [r B / R, (r + 1) B / R) in order with the loads of 16
// splits issued before their adds, then the R sums in the order r = 0 .. R-1.
// Neighbouring lanes take neighbouring slots, so reads are coalesced.  The
// bound of a small active set is the chain of dependent round trips to L2,
// which R lanes cut R-fold.  With the evaluation's ForceWork, only the splits
// that hold sources of the slot's cluster are read (the evaluation's splits
// are whole units of nt sources), and a slot whose particle is out of range,
// which the evaluation skipped, is not written.
template <int R>
__global__ __launch_bounds__(256) void reduce_split(const double *part, int32_t B,
                                                    int64_t n_act, ForceOut out, ForceWork w,
                                                    const int32_t *cluster_of, int nt)
{
    constexpr int S = 256 / R;   // sums per workgroup
    __shared__ double ps[R][S];
    const int kl = threadIdx.x % S, rl = threadIdx.x / S;
    const int64_t t = (int64_t)blockIdx.x * S + kl;
    const bool in = t < n_act * 10;
    const int q = (int)(t / n_act);
    const int64_t k = t - (int64_t)q * n_act;
    double r = 0.0;
    bool valid = in;
    if (in) {
        const int64_t i = w.idx ? (int64_t)w.idx[k] : k;
        valid = i >= 0 && i < (w.n_src > 0 ? w.n_src : w.off[w.nc]);
        if (w.n_src > 0) {
            B = (int32_t)splits_used(w.n_src, B, nt);
        } else {
            const int c = cluster_of && valid ? cluster_of[i] : 0;
            B = (int32_t)splits_used(w.off[c + 1] - w.off[c], B, nt);
        }
        const int64_t stride = 10 * n_act;
        const int b0 = (int)((int64_t)rl * B / R), b1 = (int)((int64_t)(rl + 1) * B / R);
        const double *p = part + (int64_t)q * n_act + k;
        constexpr int U = 16;
        int b = b0;
        for (; b + U <= b1; b += U) {
            double v[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                v[u] = p[(int64_t)(b + u) * stride];
#pragma unroll
            for (int u = 0; u < U; ++u)
                r += v[u];
        }
        for (; b < b1; ++b)
            r += p[(int64_t)b * stride];
    }
    if constexpr (R > 1) {
        ps[rl][kl] = r;
        __syncthreads();
        r = ps[0][kl];
#pragma unroll
        for (int u = 1; u < R; ++u)
            r += ps[u][kl];
    }
    if (!valid || rl != 0)
        return;
    if (q == 9) {
        if (out.pot)
            out.pot[k] = r;
    } else {
        out.vec[q / 3][k * out.sk + (q % 3) * out.sd] = r;
    }
}

// R by the length of the chains: 16 loads in flight per lane.  Sums that fill
// the chip by themselves (2^16 of them and more) take one lane each.
void launch_reduce(const double *part, int32_t B, int64_t n_act, const ForceOut &out,
                   const ForceWork &w, const int32_t *cluster_of, int nt, hipStream_t s)
{
    const int64_t sums = n_act * 10;
    const int R = B <= 16 || sums >= (int64_t(1) << 16) ? 1 : (B <= 64 ? 4 : 8);
    const auto k = R == 1 ? reduce_split<1> : (R == 4 ? reduce_split<4> : reduce_split<8>);
    hipLaunchKernelGGL(k, dim3((unsigned)((sums * R + 255) / 256)), dim3(256), 0, s, part, B,
                       n_act, out, w, cluster_of, nt);
}

// ---- dispatch table over the template parameters
template <typename R>
using KForce = void (*)(R, ForceWork, ForceOut, double *, int64_t, double);

// Two active particles per lane group are built for 1, 2 and 4 lanes per
// particle (the large active sets, where the LDS reads per pair matter);
// smaller sets use one.
template <int PREC, bool EPS0, int NW, bool PHI>
auto pick_lpi(int lpi_log2, int ipt)
{
    using K = KForce<SrcOf<PREC, PHI>>;
    static const K tab[7] = {
        force_kernel<PREC, 1, NW, EPS0, PHI, 1>,  force_kernel<PREC, 2, NW, EPS0, PHI, 1>,
        force_kernel<PREC, 4, NW, EPS0, PHI, 1>,  force_kernel<PREC, 8, NW, EPS0, PHI, 1>,
        force_kernel<PREC, 16, NW, EPS0, PHI, 1>, force_kernel<PREC, 32, NW, EPS0, PHI, 1>,
        force_kernel<PREC, 64, NW, EPS0, PHI, 1>};
    static const K tab2[3] = {force_kernel<PREC, 1, NW, EPS0, PHI, 2>,
                              force_kernel<PREC, 2, NW, EPS0, PHI, 2>,
                              force_kernel<PREC, 4, NW, EPS0, PHI, 2>};
    return ipt == 2 && lpi_log2 <= 2 ? tab2[lpi_log2] : tab[lpi_log2];
}

template <int PREC, bool EPS0, bool PHI>
auto pick_kernel(int lpi_log2, int nw, int ipt = 1)
{
    if (nw == 1)
        return pick_lpi<PREC, EPS0, 1, PHI>(lpi_log2, ipt);
    if (nw == 2)
        return pick_lpi<PREC, EPS0, 2, PHI>(lpi_log2, ipt);
    return pick_lpi<PREC, EPS0, 4, PHI>(lpi_log2, ipt);
}

// launch of the kernel for a shape, softening and outputs
template <int PREC, bool PHI>
void launch_variant(const SrcOf<PREC, PHI> &J, bool eps0, const Launch &L, int lpi_log2, dim3 grid,
                    const ForceWork &w, const ForceOut &out, double *part, int64_t n_act,
                    double eps2, hipStream_t s)
{
    const auto k = eps0 ? pick_kernel<PREC, true, PHI>(lpi_log2, L.waves, L.ipt)
                        : pick_kernel<PREC, false, PHI>(lpi_log2, L.waves, L.ipt);
    hipLaunchKernelGGL(k, grid, dim3(64 * L.waves), 0, s, J, w, out, part, n_act, eps2);
}

int ilog2(int64_t v)
{
    int r = 0;
    while ((int64_t(1) << (r + 1)) <= v)
        ++r;
    return r;
}

}  // namespace

int64_t iblock_size(const Launch &L) { return (int64_t)L.waves * (64 / L.lpi) * L.ipt; }

// Launch shape: the pinned one, else the autotuner's for this power of two
// of N_act, else a rule (below).
Launch pick_launch(const Ctx &c, int64_t n_act, int64_t n_src)
{
    if (c.pinned.lpi > 0)
        return c.pinned;
    if (n_act >= 1 && !c.tuned.empty()) {
        const int b = ilog2(n_act);
        if (b < (int)c.tuned.size() && c.tuned[b].lpi > 0) {
            Launch L = c.tuned[b];
            // at least one tile per split of the largest source range, and
            // the partials within the split buffer
            while (L.split > 1 && ((int64_t)L.split * n_act > c.part_cap ||
                                   n_src / L.split < 64 * L.waves))
                L.split >>= 1;
            return L;
        }
    }
    return rule_launch(n_act, n_src, c.part_cap, c.cfg.precision);
}

// Launch rule.  4 waves; about 4096 lanes per split (lanes per particle
// 4096 / N_act, between 1 and 64); two particles per lane group for active
// sets of 2^15 and more in the modes with FP64 pair arithmetic (it halves
// the LDS reads per pair: 1-3 % faster there, measured; the FP32-pair mode
// is faster with one).  Then the sources are split:
//   - up to 4096 workgroups while every split keeps a tile: the chip holds
//     768-1024 at once, and with several rounds of them a compute unit that
//     is done takes the next.  Against the earlier limit of 2048 with two
//     tiles per split: 7424 active x 32,768 sources 480 -> 436 us (64 -> 128
//     splits), 2176 x 32,768 172 -> 148 us, 23,296 x 32,768 1387 -> 1357 us
//     (16 -> 32); more do not help, and add partial sums;
//   - with 16 or more lanes per particle and a split of few tiles, up to 1792
//     workgroups while every split keeps two tiles: a workgroup's start, lane
//     sums and partial results then weigh as much as its pairs, so one round
//     is best: 64 active x 65,536 sources 20.2 + 4.1 us (evaluation + split
//     sums) with 64 splits, 22.7 + 6.2 us with 128, 22.2 + 4.0 us with 32;
//   - for large source sets further while every split holds 2^17 sources: a
//     split's work dwarfs its partials' traffic there.  65,536 active x
//     8,388,608 sources: split 16 / 32 / 64 / 128 / 256 -> 946 / 935 / 930 /
//     927 / 925 ms, but 3.4 / 4.5 / 6.8 / 11.2 / 20.2 GB fetched (shorter
//     walks, started at staggered times, share the L2 less); 2^17 stops at 64.
// Powers of two only: some other splits of a particle pair per lane group
// measured up to 16 % slower (65,536 x 65,536: 16 splits 7.50 ms, 18 8.74 ms).
Launch rule_launch(int64_t n_act, int64_t n_src, int64_t part_cap, int prec)
{
    Launch L;
    L.waves = 4;
    L.lpi = 1;
    L.split = 1;
    while (n_act * L.lpi < 4096 && L.lpi < 64)
        L.lpi <<= 1;
    L.ipt = prec != NBODY_PREC_FP32PAIR && L.lpi <= 4 && n_act * L.lpi >= (int64_t(1) << 15) ? 2 : 1;
    const int64_t nt = 64 * L.waves;
    const int64_t long_split = int64_t(1) << 17;
    const int64_t n_ib = (n_act + iblock_size(L) - 1) / iblock_size(L);
    for (;;) {
        const int64_t b2 = (int64_t)L.split * 2, per_split = n_src / b2;
        const bool latency = L.lpi >= 16 && per_split < 16 * nt;
        if (per_split < (latency ? 2 : 1) * nt || b2 * n_act > part_cap || b2 > 65535)   // grid y limit
            break;
        if (n_ib * b2 > (latency ? 1792 : 4096) && per_split < long_split)
            break;
        L.split <<= 1;
    }
    return L;
}

hipError_t launch_force(Ctx &c, const ForceWork &w, const Launch &L,
                        const ForceOut &out, int64_t n_act_total, hipStream_t s, bool reduce,
                        bool staged)
{
    if (n_act_total <= 0 || w.n_blocks <= 0)
        return hipSuccess;
    const int lg = ilog2(L.lpi);
    const bool eps0 = c.eps == 0.0;
    const double eps2 = c.eps * c.eps;
    double *part = w.split > 1 || staged ? c.part : nullptr;
    // one cluster: no workgroups for splits without sources
    const int64_t gy = w.blk_cluster ? w.split
                                     : splits_used(w.n_src, w.split, split_unit(L.lpi, L.waves));
    const dim3 grid((unsigned)w.n_blocks, (unsigned)gy);
    const int prec = c.cfg.precision;
    const bool phi = out.pot != nullptr;   // potential wanted (not in block steps)
    const int rec = prof_begin(c, PH_FORCE, n_act_total);
    auto go = [&](auto p, const auto &packed) {
        constexpr int P = decltype(p)::value;
        if (phi)
            launch_variant<P, true>(c.js, eps0, L, lg, grid, w, out, part, n_act_total, eps2, s);
        else
            launch_variant<P, false>(packed, eps0, L, lg, grid, w, out, part, n_act_total, eps2, s);
    };
    if (prec == NBODY_PREC_MIXED)
        go(std::integral_constant<int, PREC_MIXED>{}, c.jm);
    else if (prec == NBODY_PREC_FP32PAIR)
        go(std::integral_constant<int, PREC_PAIR32>{}, c.jp);
    else
        go(std::integral_constant<int, PREC_F64>{}, c.jd);
    prof_end(c, rec);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !part || !reduce)
        return e;
    const int rr = prof_begin(c, PH_REDUCE);
    launch_reduce(c.part, w.split, n_act_total, out, w, c.d_cluster_of,
                  split_unit(L.lpi, L.waves), s);
    prof_end(c, rr);
    return hipGetLastError();
}

// Potential of the stored state for the energy: split b's part of
// phi[i] = -sum over the particle's half-window of m_j / r_ij (every pair of a
// cluster once) to c.part[b n + i], or to c.d_phi[i] when *split is 1.
hipError_t launch_energy_pot(Ctx &c, int *split, const double **phi, hipStream_t s)
{
    const int64_t n = c.n;
    const ClusterSizes &z = c.sizes;
    const int64_t ncmax = z.largest;
    // Two particles per lane from 32,768 bodies (below, they leave too few
    // workgroups: 24,000 bodies 239 us, one 216; 40,000 425 and 440; 100,003
    // 2276 and 2377; four 2407, and nowhere better up to 2^20), unless small
    // clusters would leave lanes without a second one: those walk their whole
    // window all the same (65,536 bodies with 2000 clusters of 256: 2.35 ms
    // with two, 1.60 with one; with three clusters of 30,000: 1.70 and 1.87).
    const int ipt = ncmax >= 32768 && 2 * z.wg2 <= z.wg1 + z.wg1 / 8 ? 2 : 1;
    const int64_t ib = 256 * ipt;
    hipError_t e = hipSuccess;
    ForceWork w{};
    w.off = c.d_off;
    w.nc = c.nc;
    w.err = c.d_err;
    if (c.nc == 1) {
        w.n_blocks = (n + ib - 1) / ib;
    } else {
        const int64_t cap = n / ib + c.nc + 1;
        if ((e = launch_segments(c, nullptr, n, s)) != hipSuccess ||
            (e = launch_blocks(c, ib, cap, s)) != hipSuccess)
            return e;
        w.blk_cluster = c.d_blk_cluster;
        w.blk_first = c.d_blk_first;
        w.n_blocks = cap;
    }
    // splits of at least a tile, up to ~8192 workgroups (several rounds of the
    // 1024-2048 resident ones: 100,003 bodies 2.31 / 2.29 / 2.28 ms with up to
    // 2048 / 4096 / 8192, 66,000 1072 / 1051 / 1032 us), and the partial sums
    // within the split buffer; of the upper half of these the number that
    // fills the 256 compute units most evenly (against the largest power of
    // two of at least two tiles: 9000 bodies 88 -> 80 us, 13,000 113 -> 98,
    // 5000 82 -> 64)
    // Several clusters: if the large ones are most of the work, the splits are
    // counted for their workgroups alone, as the small ones' few tiles leave
    // the chip to a few long walks (40,000 bodies with 3000 clusters of 100,
    // split 1 / 2 / 4 / 8 / 16 / 20: 913 / 841 / 1106 / 688 / 622 / 605 us);
    // not otherwise (65,536 with 10,000 of 256, which are 38 % of the pairs:
    // split 1 1826 us, 20 2075).
    const int64_t wgs = c.nc > 1 && z.big_share >= 0.75 ? std::max<int64_t>(1, z.wg_big / ipt) : w.n_blocks;
    int64_t most = std::min<int64_t>(8192 / wgs, (ncmax / 2 + ib) / 256);
    most = std::max<int64_t>(1, std::min<int64_t>(most, 10 * c.part_cap / n));
    *split = (int)most;
    double best = 0.0;
    for (int64_t k = most; k > most / 2; --k) {
        const double rounds = (double)(wgs * k) / 256.0, even = rounds / std::ceil(rounds);
        if (even > best + 0.01) {
            best = even;
            *split = (int)k;
        }
    }
    w.split = *split;
    const double *X = c.st.pos, *Y = c.st.pos + n, *Z = c.st.pos + 2 * n;
    double *dst = *split > 1 ? c.part : c.d_phi;
    *phi = dst;
    const float e2 = (float)(c.eps * c.eps);
    auto pick = [&](auto none, auto normal, auto odd) {
        return c.eps == 0.0 ? none : (std::isnormal(e2) ? normal : odd);
    };
    const auto k =
        ipt == 2
            ? pick(energy_kernel<EPS_NONE, 2>, energy_kernel<EPS_NORMAL, 2>, energy_kernel<EPS_ODD, 2>)
            : pick(energy_kernel<EPS_NONE, 1>, energy_kernel<EPS_NORMAL, 1>, energy_kernel<EPS_ODD, 1>);
    const int rec = prof_begin(c, PH_ENERGY);
    hipLaunchKernelGGL(k, dim3((unsigned)w.n_blocks, (unsigned)*split), dim3(256), 0, s, X, Y, Z,
                       (const double *)c.st.mass, w, dst, n, c.eps * c.eps);
    prof_end(c, rec);
    return hipGetLastError();
}

}  // namespace nb
