// Evaluation step of the Hermite scheme (paper Sect. 3, item 2, with the
// softened potential of Sect. 2): the per-workgroup body shared by the
// launch kernel (force.hip) and the device-resident block-step loop
// (integrate.hip).  The design notes are at the top of force.hip.
#pragma once
#include "nbody_internal.h"

namespace nb {

namespace {

// kernel variants: the two public mixed modes and the FP64 path
constexpr int PREC_MIXED = 0, PREC_F64 = 1, PREC_PAIR32 = 4;

// Accesses to data that the workgroups of a persistent launch exchange.  COH:
// single accesses that are coherent over the device (relaxed atomics at agent
// scope), so that a barrier between the workgroups needs only to wait for
// them, not to write back and invalidate the XCDs' L2 caches; otherwise plain
// ones (data of other launches, or of one workgroup).
template <bool COH, typename T>
__device__ __forceinline__ T ld(const T *p)
{
    if constexpr (COH)
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        return *p;
}
template <bool COH, typename T>
__device__ __forceinline__ void put(T *p, T v)
{
    if constexpr (COH)
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        *p = v;
}

// Knuth's two-sum: (hi, lo) += p without rounding loss in the (hi, lo) pair.
__device__ __forceinline__ void ds_add(float &hi, float &lo, float p)
{
    const float s = hi + p;
    const float bp = s - hi;
    const float e = (hi - (s - bp)) + (p - bp);
    hi = s;
    lo += e;
}

// Far-away, massless stand-in for source slots past the end of a range.
constexpr double NULL_POS = 1.0e15;

template <int PREC>
struct Smem;

template <>
struct Smem<PREC_MIXED> {
    using R = JRecMixed;
};
template <>
struct Smem<PREC_PAIR32> {
    using R = JRecPair32;
};
template <>
struct Smem<PREC_F64> {
    using R = JRecF64;
};

// 1/sqrt(r2) for the mixed path: FP32 seed from v_rsq_f32 (|error| < 1 ulp,
// measured) and one Newton step in FP64, which squares the relative error
// (~1e-14).  Used for the acceleration and potential terms and, with the
// same operations, for the removal of the j == i potential term.
__device__ __forceinline__ double rinv_mixed(double r2)
{
    const double y0 = (double)__builtin_amdgcn_rsqf((float)r2);
    const double res = fma(-r2 * y0, y0, 1.0);   // 1 - r2 y0^2
    return fma(0.5 * y0, res, y0);
}

// 1/sqrt(r2) to FP64 accuracy for the FP64 passes: the same FP32 seed y0
// (relative error |d| below ~2e-7 with the rounding of r2 to FP32), then the
// third-order step y0 (1 + e/2 + 3e^2/8), e = 1 - r2 y0^2 = O(2d), whose
// truncation error (5/16) e^3 is far below an FP64 ulp; the result is within
// about one ulp.  Valid while r2 is a normal FP32 number (r from ~1e-19 to
// ~1e19), which the softened distances of every supported system are.
__device__ __forceinline__ double rinv_f64(double r2)
{
    const double y0 = (double)__builtin_amdgcn_rsqf((float)r2);
    const double e = fma(-r2 * y0, y0, 1.0);
    return fma(y0 * e, fma(e, 0.375, 0.5), y0);
}

// v of another lane by a data-parallel-primitive move of each half
template <int CTRL>
__device__ __forceinline__ double dpp_of(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// Sums over the lanes STEP (16 or 32) apart of two values at once: the even
// rows (lower half) get a's sum, the odd rows (upper half) b's.  The swap
// leaves a and b's even parts in one register and their odd parts in the other.
template <int STEP>
__device__ __forceinline__ double swap_sum(double a, double b)
{
    const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
    double r[2];
    if constexpr (STEP == 16) {
        const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
        for (int k = 0; k < 2; ++k)
            r[k] = __longlong_as_double((long long)((uint64_t)h[k] << 32 | l[k]));
    } else {
        const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
        for (int k = 0; k < 2; ++k)
            r[k] = __longlong_as_double((long long)((uint64_t)h[k] << 32 | l[k]));
    }
    return r[0] + r[1];
}

// Sum over groups of LPI <= 32 neighbouring lanes, on every lane of the group
// and with the bits of a xor butterfly (at the steps of 4 and 8 a mirror of 8
// or 16 lanes meets the same partial sums, which are alike in a quad or half
// row by then).  Register moves only: the same sum through LDS permutes was
// a fifth of a small block's evaluation.
template <int LPI>
__device__ __forceinline__ double lane_sum(double v)
{
    if constexpr (LPI >= 2)
        v += dpp_of<0xB1>(v);    // quad_perm 1 0 3 2
    if constexpr (LPI >= 4)
        v += dpp_of<0x4E>(v);    // quad_perm 2 3 0 1
    if constexpr (LPI >= 8)
        v += dpp_of<0x141>(v);   // row_half_mirror
    if constexpr (LPI >= 16)
        v += dpp_of<0x140>(v);   // row_mirror
    if constexpr (LPI >= 32)
        v = swap_sum<16>(v, v);
    return v;
}

// The ten sums Q of a lane group (32 or 64 lanes) spread over its rows of 16
// lanes: v[k] of a lane in row r ends as the sum of quantity lane_quantity(k,
// r).  Two values share each register move of the first one or two steps, so
// the whole takes 60-75 instructions instead of 270 (64 lanes, one value at a
// time), a sixth of what a wave of a small block executes in all.  (Not in the
// ensemble loop, where it measured 2 % slower: its registers are full.)
template <int LPI>
struct LaneSums {
    static constexpr int N = LPI == 64 ? 3 : 5;
    double v[N];
    __device__ __forceinline__ LaneSums(const double *Q)
    {
        double p[5];
#pragma unroll
        for (int k = 0; k < 5; ++k)
            p[k] = swap_sum<LPI == 64 ? 32 : 16>(Q[2 * k], Q[2 * k + 1]);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            if constexpr (LPI == 64)
                v[k] = k < 2 ? swap_sum<16>(p[2 * k], p[2 * k + 1]) : swap_sum<16>(p[4], p[4]);
            else
                v[k] = p[k];
            v[k] = lane_sum<16>(v[k]);
        }
    }
    // quantity of v[k] in the group's row r (-1: held by another row)
    static __device__ __forceinline__ int quantity(int k, int r)
    {
        if (LPI == 32)
            return 2 * k + r;
        return k < 2 ? 4 * k + 2 * (r & 1) + (r >> 1) : ((r & 1) ? -1 : 8 + (r >> 1));
    }
};

// LDS tile of NT source records, one 16-byte aligned record per source
// (its fields side by side): with one lane per particle every lane reads
// the same record, and from one address every field is an immediate offset
// (with one array per field the compiler formed each field's address apart
// and copied it into a vector register per read: 2-5 % more VALU
// instructions per pair).  One tile per (precision, tile size): every
// launch shape with that tile size uses the same LDS, so a kernel that runs
// several shapes (the ensemble loop) holds one tile.
template <int PREC, int NT>
struct SrcTile {
    static constexpr bool P32 = PREC == PREC_PAIR32, MIXED = PREC == PREC_MIXED;
    using VV = typename std::conditional<P32, float, double>::type;
    using VA = typename std::conditional<MIXED || P32, float, double>::type;
    struct alignas(16) S {
        double x, y, z, m;
        VV vx, vy, vz;
        VA ax, ay, az;
    };
    S s[NT];
};

template <int PREC, int NT>
__device__ __forceinline__ SrcTile<PREC, NT> &src_tile()
{
    __shared__ SrcTile<PREC, NT> t;
    return t;
}

// The stored state of particle i that its prediction reads, and the Taylor
// series of paper Sect. 3 item 1 (Horner form) to h later.
struct PredIn {
    double x[3], v[3], a[3], j[3], s[3], c[3], m, t;
};
struct Predicted {
    double x[3], v[3], a[3];
};

template <bool COH = false>
__device__ __forceinline__ PredIn load_pred(const State &st, int64_t n, int64_t i)
{
    PredIn q;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int64_t e = (int64_t)d * n + i;
        q.x[d] = ld<COH>(st.pos + e);
        q.v[d] = ld<COH>(st.vel + e);
        q.a[d] = ld<COH>(st.acc + e);
        q.j[d] = ld<COH>(st.jrk + e);
        q.s[d] = ld<COH>(st.snp + e);
        q.c[d] = ld<COH>(st.crk + e);
    }
    q.m = st.mass[i];
    q.t = ld<COH>(st.t + i);
    return q;
}

__device__ __forceinline__ Predicted predict(const PredIn &q, double h)
{
    Predicted p;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double x = q.x[d], v = q.v[d], a = q.a[d];
        const double j = q.j[d], s = q.s[d], c = q.c[d];
        p.x[d] = x + h * (v + h * (a * 0.5 + h * (j * (1.0 / 6) + h * (s * (1.0 / 24) + h * (c * (1.0 / 120))))));
        p.v[d] = v + h * (a + h * (j * 0.5 + h * (s * (1.0 / 6) + h * (c * (1.0 / 24)))));
        p.a[d] = a + h * (j + h * (s * 0.5 + h * (c * (1.0 / 6))));
    }
    return p;
}

// Sources predicted on the way to LDS: the state of a system of n particles
// advanced to T, the active particles' indices from src0 in an LDS list.
struct JState {
    const State *st;
    int64_t n;
    double T;
    const uint16_t *list;
};

// Distance between neighbouring particles of a source array
template <typename R>
__device__ __forceinline__ constexpr int64_t rec_stride(const R &)
{
    return 1;
}
__device__ __forceinline__ int64_t rec_stride(const JSrc &J) { return J.st; }
__device__ __forceinline__ int64_t rec_stride(const JState &) { return 1; }

// One workgroup's share of an evaluation: i-block g (IB active slots) against
// source split b.  J: packed records of the precision, or the FP64 sources as
// they stand (JSrc) or predicted (JState), rounded to the record's types on
// the way to LDS.  The launch kernel calls it with (blockIdx.x, blockIdx.y);
// the device-resident block-step loop calls it for the units it takes.
// Every early return is uniform over the workgroup.  PHI: also sum the
// potential (nbody_force); a block step's evaluation
// does not need it (the energy has its own pass).  IPT: active particles
// per lane group (each source read from LDS serves IPT pairs).
template <int PREC, int LPI, int NW, bool EPS0, bool PHI, int IPT = 1, bool AHEAD = true,
          bool COH = false, typename R>
__device__ __forceinline__ void force_block(const R &J, const ForceWork &w, const ForceOut &out,
                                            double *part, int64_t n_act_total, double eps2,
                                            int64_t g, int b)
{
    constexpr int NT = NW * 64;      // sources per LDS tile
    constexpr int GI = 64 / LPI;     // lane groups (of LPI lanes) per wave
    constexpr int NG = NW * GI;      // lane groups per workgroup
    constexpr int IB = NG * IPT;     // active particles per workgroup
    constexpr int PER = NT / LPI;    // sources per lane per tile
    // pairs per lane of one FP32 partial sum: a short one keeps its rounding
    // small (64 pairs measured 3x better than 256 for FP32 jerk sums, at ~1%
    // more instructions)
    constexpr int FOLD = PER < 64 ? PER : 64;
    static_assert(FOLD * LPI == split_unit(LPI, NW), "unit of a split");
    constexpr bool MIXED = PREC == PREC_MIXED;
    constexpr bool P32 = PREC == PREC_PAIR32;
    constexpr int NV = 9;            // vector outputs (a, da, d2a)
    // FP32 accumulators (mixed: snap; FP32-pair mode: all nine); FP64 ones
    // for the rest
    constexpr int NF = MIXED ? 3 : (P32 ? 9 : 1);
    constexpr int ND = MIXED ? 6 : (P32 ? 1 : NV);
    // types of the sources' velocity and acceleration (as in the records)
    using VV = typename std::conditional<P32, float, double>::type;
    using VA = typename std::conditional<MIXED || P32, float, double>::type;

    SrcTile<PREC, NT> &tl = src_tile<PREC, NT>();

    // ---- which active slots and which sources this workgroup takes
    int64_t gfirst = 0, s0 = 0, s1 = w.n_act, o0 = w.src0, o1 = w.src0 + w.n_src;
    if (w.blk_cluster) {
        const int c = w.blk_cluster[g];
        if (c < 0)
            return;  // grid padding past the last i-block
        gfirst = w.blk_first[c];
        s0 = w.seg[c];
        s1 = w.seg[c + 1];
        o0 = w.off[c];
        o1 = w.off[c + 1];
    }
    const int64_t kb = s0 + (g - gfirst) * IB;
    // splits past this cluster's sources (splits are whole units, so a small
    // cluster fills fewer than B of them): nothing to do, and the reduction
    // reads only the splits in use
    const int64_t used = splits_used(o1 - o0, w.split, FOLD * LPI);
    if (b >= used)
        return;
    const int64_t j0 = o0 + split_begin(o1 - o0, used, FOLD * LPI, b);
    const int64_t j1 = o0 + split_begin(o1 - o0, used, FOLD * LPI, b + 1);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int il = wave * GI + lane / LPI;   // lane group
    const int js = lane & (LPI - 1);         // slot within the group
    // The record of this lane's source of tile t0, in registers.  Each tile
    // is fetched one tile ahead: the first before the active particles (two
    // dependent loads), the others while the tile before is evaluated.  A
    // small active set has only a few tiles per workgroup, and their load
    // latencies (1-2 us each, behind the launch's) were most of its time.
    // Not with AHEAD false: the ensemble loop's four waves per SIMD have no
    // registers left for it (7 % slower there, spilling).
    using Rec = typename SrcTile<PREC, NT>::S;
    const int64_t st = rec_stride(J);
    auto fetch = [&](int64_t t0) {
        Rec r;
        // past the range: the last source, without mass
        const int64_t jt = t0 + tid, jj = jt < j1 ? jt : j1 - 1, e = jj * st;
        if constexpr (std::is_same<R, JState>::value) {
            const PredIn q = load_pred<COH>(*J.st, J.n, jj);
            const Predicted p = predict(q, J.T - q.t);
            r.x = p.x[0]; r.y = p.x[1]; r.z = p.x[2];
            r.m = jt < j1 ? q.m : 0.0;
            r.vx = (VV)p.v[0]; r.vy = (VV)p.v[1]; r.vz = (VV)p.v[2];
            r.ax = (VA)p.a[0]; r.ay = (VA)p.a[1]; r.az = (VA)p.a[2];
            return r;
        } else {
        r.x = ld<COH>(J.x + e); r.y = ld<COH>(J.y + e); r.z = ld<COH>(J.z + e);
        r.m = ld<COH>(J.m + jj);
        r.vx = (VV)ld<COH>(J.vx + e); r.vy = (VV)ld<COH>(J.vy + e); r.vz = (VV)ld<COH>(J.vz + e);
        r.ax = (VA)ld<COH>(J.ax + e); r.ay = (VA)ld<COH>(J.ay + e); r.az = (VA)ld<COH>(J.az + e);
        if constexpr (!P32)
            r.m = jt < j1 ? r.m : 0.0;
        return r;
        }
    };
    Rec next;
    if constexpr (AHEAD)
        next = fetch(j0);
    // particle u of the lane group: active slot kb + il + u NG
    int64_t k[IPT], i[IPT];
    bool valid[IPT];
    double xi[IPT], yi[IPT], zi[IPT];
    VV vxi[IPT], vyi[IPT], vzi[IPT];
    VA axi[IPT], ayi[IPT], azi[IPT];
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
        k[u] = kb + il + u * NG;
        valid[u] = k[u] < s1;
        const int64_t kk = valid[u] ? k[u] : kb;
        if constexpr (std::is_same<R, JState>::value)
            i[u] = o0 + J.list[kk];
        else
            i[u] = w.idx ? (int64_t)ld<COH>(w.idx + kk) : kk;
        if (i[u] < o0 || i[u] >= o1) {
            // an index outside its cluster (a caller's bad list): skip the
            // slot, load a valid particle, report
            if (valid[u] && js == 0 && w.err)
                atomicOr(w.err, ERR_BADIDX);
            valid[u] = false;
            i[u] = o0;
        }
        if constexpr (std::is_same<R, JState>::value) {
            const PredIn q = load_pred<COH>(*J.st, J.n, i[u]);
            const Predicted p = predict(q, J.T - q.t);
            xi[u] = p.x[0]; yi[u] = p.x[1]; zi[u] = p.x[2];
            vxi[u] = (VV)p.v[0]; vyi[u] = (VV)p.v[1]; vzi[u] = (VV)p.v[2];
            axi[u] = (VA)p.a[0]; ayi[u] = (VA)p.a[1]; azi[u] = (VA)p.a[2];
            continue;
        } else {
        const int64_t e = i[u] * st;
        xi[u] = ld<COH>(J.x + e); yi[u] = ld<COH>(J.y + e); zi[u] = ld<COH>(J.z + e);
        vxi[u] = (VV)ld<COH>(J.vx + e); vyi[u] = (VV)ld<COH>(J.vy + e);
        vzi[u] = (VV)ld<COH>(J.vz + e);
        axi[u] = (VA)ld<COH>(J.ax + e); ayi[u] = (VA)ld<COH>(J.ay + e);
        azi[u] = (VA)ld<COH>(J.az + e);
        }
    }

    // the active particles' values are in registers from here on: without
    // this the wait for their loads lands in the pair loop, where it also
    // waits for the next tile's
#pragma unroll
    for (int u = 0; u < (AHEAD ? IPT : 0); ++u)
        asm volatile("" : "+v"(xi[u]), "+v"(yi[u]), "+v"(zi[u]), "+v"(vxi[u]), "+v"(vyi[u]),
                     "+v"(vzi[u]), "+v"(axi[u]), "+v"(ayi[u]), "+v"(azi[u]));

    // FP64 sums (mixed: acceleration and jerk; FP64 passes: everything),
    // the potential in FP64 always, and double-single (hi, lo) pairs for
    // the FP32 sums (mixed: snap; FP32-pair mode: everything), fed by FP32
    // partial sums over at most FOLD pairs per lane
    double D[IPT][ND];
    float H[IPT][NF], L[IPT][NF];
    double phi[IPT];
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
#pragma unroll
        for (int q = 0; q < ND; ++q)
            D[u][q] = 0.0;
#pragma unroll
        for (int q = 0; q < NF; ++q) {
            H[u][q] = 0.0f;
            L[u][q] = 0.0f;
        }
        phi[u] = 0.0;
    }

    for (int64_t t0 = j0; t0 < j1; t0 += NT) {
        __syncthreads();
        if constexpr (!AHEAD)
            next = fetch(t0);
        if constexpr (P32) {
            // Field by field: a copy of the whole record also writes its eight
            // bytes of padding, in unaligned pieces.  The mass past the range
            // is dropped here and not in the fetch, which would wait for the
            // mass there: 32 active of 524,288 sources 70.9 -> 57.4 us (the
            // other modes' records have no such padding, and the pair loop
            // that the compiler then makes of them is 1 % slower on the
            // largest sets: 117.9 -> 118.9 ms with the potential).
            auto &to = tl.s[tid];
            to.x = next.x; to.y = next.y; to.z = next.z;
            to.m = t0 + tid < j1 ? next.m : 0.0;
            to.vx = next.vx; to.vy = next.vy; to.vz = next.vz;
            to.ax = next.ax; to.ay = next.ay; to.az = next.az;
        } else {
            tl.s[tid] = next;
        }
        __syncthreads();
        if constexpr (AHEAD)
            if (t0 + NT < j1)
                next = fetch(t0 + NT);

        // the last tile of a walk may hold fewer units than a whole one
        const int pend = t0 + NT <= j1 ? PER : (int)((j1 - t0 + LPI - 1) / LPI);
        for (int p0 = 0; p0 < pend; p0 += FOLD) {
            float T[IPT][NF];
#pragma unroll
            for (int u = 0; u < IPT; ++u)
#pragma unroll
                for (int q = 0; q < NF; ++q)
                    T[u][q] = 0.0f;

            constexpr int UNROLL = PER > 16 ? (IPT == 1 ? 4 : 2) : (AHEAD ? 1 : 4);
#pragma unroll UNROLL
            for (int p = p0; p < p0 + FOLD; ++p) {
                const int t = js + p * LPI;
                const auto &sr = tl.s[t];
                const double sx = sr.x, sy = sr.y, sz = sr.z, sm = sr.m;
                const VV svx = sr.vx, svy = sr.vy, svz = sr.vz;
                const VA sax = sr.ax, say = sr.ay, saz = sr.az;
#pragma unroll
                for (int u = 0; u < IPT; ++u) {
                    if constexpr (P32) {
                        // every pair term in FP32 from the FP64 difference r_j - r_i
                        const float dx = (float)(sx - xi[u]), dy = (float)(sy - yi[u]),
                                    dz = (float)(sz - zi[u]);
                        const float r2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, (float)eps2)));
                        float rinv = __builtin_amdgcn_rsqf(r2);
                        if constexpr (EPS0)
                            rinv = r2 > 0.0f ? rinv : 0.0f;
                        const float mrinv = (float)sm * rinv;
                        if constexpr (PHI)
                            phi[u] -= (double)mrinv;
                        const float rinv2 = rinv * rinv, mr3 = mrinv * rinv2;
                        const float dvx = svx - vxi[u], dvy = svy - vyi[u], dvz = svz - vzi[u];
                        const float dax = sax - axi[u], day = say - ayi[u], daz = saz - azi[u];
                        const float rv = fmaf(dx, dvx, fmaf(dy, dvy, dz * dvz));
                        const float qq = fmaf(dvx, dvx, fmaf(dvy, dvy, fmaf(dvz, dvz,
                                         fmaf(dx, dax, fmaf(dy, day, dz * daz)))));
                        const float alpha = rv * rinv2;
                        const float beta = fmaf(alpha, alpha, qq * rinv2);
                        const float a3 = -3.0f * alpha, a6 = a3 + a3, b3 = -3.0f * beta;
                        const float jx = fmaf(a3, dx, dvx), jy = fmaf(a3, dy, dvy),
                                    jz = fmaf(a3, dz, dvz);
                        float *Tu = T[u];
                        Tu[0] = fmaf(mr3, dx, Tu[0]);
                        Tu[1] = fmaf(mr3, dy, Tu[1]);
                        Tu[2] = fmaf(mr3, dz, Tu[2]);
                        Tu[3] = fmaf(mr3, jx, Tu[3]);
                        Tu[4] = fmaf(mr3, jy, Tu[4]);
                        Tu[5] = fmaf(mr3, jz, Tu[5]);
                        Tu[6] = fmaf(mr3, fmaf(a6, jx, fmaf(b3, dx, dax)), Tu[6]);
                        Tu[7] = fmaf(mr3, fmaf(a6, jy, fmaf(b3, dy, day)), Tu[7]);
                        Tu[8] = fmaf(mr3, fmaf(a6, jz, fmaf(b3, dz, daz)), Tu[8]);
                        continue;
                    }
                    const double dxd = sx - xi[u], dyd = sy - yi[u], dzd = sz - zi[u];
                    const double r2 = fma(dxd, dxd, fma(dyd, dyd, fma(dzd, dzd, eps2)));
                    double rinv;
                    if constexpr (MIXED)
                        rinv = rinv_mixed(r2);
                    else
                        rinv = rinv_f64(r2);
                    if constexpr (EPS0)
                        rinv = r2 > 0.0 ? rinv : 0.0;
                    const double mrinv = sm * rinv;
                    if constexpr (PHI)
                        phi[u] -= mrinv;
                    const double rinv2 = rinv * rinv;
                    const double mr3 = mrinv * rinv2;
                    double *Du = D[u];
                    if constexpr (MIXED) {
                        // acceleration and jerk in FP64, snap in FP32:
                        // A = m r^-3 r, J = m r^-3 (v - 3 alpha r),
                        // S = m r^-3 (a - 6 alpha jv - 3 beta r), jv = v - 3 alpha r
                        Du[0] = fma(mr3, dxd, Du[0]);
                        Du[1] = fma(mr3, dyd, Du[1]);
                        Du[2] = fma(mr3, dzd, Du[2]);
                        const double dvx = svx - vxi[u], dvy = svy - vyi[u], dvz = svz - vzi[u];
                        const double m3r2 = -3.0 * rinv2;
                        const double a3d = fma(dxd, dvx, fma(dyd, dvy, dzd * dvz)) * m3r2;  // -3 alpha
                        const double jxd = fma(a3d, dxd, dvx), jyd = fma(a3d, dyd, dvy),
                                     jzd = fma(a3d, dzd, dvz);
                        Du[3] = fma(mr3, jxd, Du[3]);
                        Du[4] = fma(mr3, jyd, Du[4]);
                        Du[5] = fma(mr3, jzd, Du[5]);
                        const float dx = (float)dxd, dy = (float)dyd, dz = (float)dzd;
                        const float fvx = (float)dvx, fvy = (float)dvy, fvz = (float)dvz;
                        const float jx = (float)jxd, jy = (float)jyd, jz = (float)jzd;
                        const float a3 = (float)a3d, f3r2 = (float)m3r2, fm3 = (float)mr3;
                        const float dax = sax - axi[u], day = say - ayi[u], daz = saz - azi[u];
                        const float qq = fmaf(fvx, fvx, fmaf(fvy, fvy, fmaf(fvz, fvz,
                                         fmaf(dx, dax, fmaf(dy, day, dz * daz)))));
                        // -3 beta = -3 alpha^2 - 3 qq / s^2, with alpha = -a3 / 3
                        const float b3 = fmaf(a3, a3 * (-1.0f / 3.0f), qq * f3r2);
                        const float a6 = a3 + a3;
                        const float sxf = fmaf(a6, jx, fmaf(b3, dx, dax));
                        const float syf = fmaf(a6, jy, fmaf(b3, dy, day));
                        const float szf = fmaf(a6, jz, fmaf(b3, dz, daz));
                        T[u][0] = fmaf(fm3, sxf, T[u][0]);
                        T[u][1] = fmaf(fm3, syf, T[u][1]);
                        T[u][2] = fmaf(fm3, szf, T[u][2]);
                    } else {
                        const double dvx = svx - vxi[u], dvy = svy - vyi[u], dvz = svz - vzi[u];
                        const double dax = sax - axi[u], day = say - ayi[u], daz = saz - azi[u];
                        const double alpha = fma(dxd, dvx, fma(dyd, dvy, dzd * dvz)) * rinv2;
                        const double qq = fma(dvx, dvx, fma(dvy, dvy, fma(dvz, dvz,
                                          fma(dxd, dax, fma(dyd, day, dzd * daz)))));
                        const double beta = fma(alpha, alpha, qq * rinv2);
                        const double a3 = -3.0 * alpha, a6 = a3 + a3, b3 = -3.0 * beta;
                        const double jx = fma(a3, dxd, dvx), jy = fma(a3, dyd, dvy),
                                     jz = fma(a3, dzd, dvz);
                        Du[0] = fma(mr3, dxd, Du[0]);
                        Du[1] = fma(mr3, dyd, Du[1]);
                        Du[2] = fma(mr3, dzd, Du[2]);
                        Du[3] = fma(mr3, jx, Du[3]);
                        Du[4] = fma(mr3, jy, Du[4]);
                        Du[5] = fma(mr3, jz, Du[5]);
                        Du[6] = fma(mr3, fma(a6, jx, fma(b3, dxd, dax)), Du[6]);
                        Du[7] = fma(mr3, fma(a6, jy, fma(b3, dyd, day)), Du[7]);
                        Du[8] = fma(mr3, fma(a6, jz, fma(b3, dzd, daz)), Du[8]);
                    }
                }
            }
            if constexpr (MIXED || P32) {
#pragma unroll
                for (int u = 0; u < IPT; ++u)
#pragma unroll
                    for (int q = 0; q < NF; ++q)
                        ds_add(H[u][q], L[u][q], T[u][q]);
            }
        }
    }

#pragma unroll
    for (int u = 0; u < IPT; ++u) {
        // ---- combine the LPI lanes of each active particle
        double Q[NV + 1];
        if constexpr (P32) {
#pragma unroll
            for (int q = 0; q < NF; ++q)
                Q[q] = (double)H[u][q] + (double)L[u][q];
        } else if constexpr (MIXED) {
#pragma unroll
            for (int q = 0; q < 6; ++q)
                Q[q] = D[u][q];
#pragma unroll
            for (int q = 0; q < NF; ++q)
                Q[6 + q] = (double)H[u][q] + (double)L[u][q];
        } else {
#pragma unroll
            for (int q = 0; q < NV; ++q)
                Q[q] = D[u][q];
        }
        Q[NV] = phi[u];
        const int64_t ku = k[u], iu = i[u];
        // the j == i pair adds exactly zero to a, da, d2a but -m_i / eps to the
        // potential: that term, computed with the same operations, to remove it
        auto self_phi = [&]() -> double {
            if (EPS0 || !PHI || iu < j0 || iu >= j1)
                return 0.0;
            if constexpr (std::is_same<R, JState>::value) {
                return 0.0;   // (no potential in block steps)
            } else if constexpr (P32) {
                const float e2f = (float)eps2;
                const float ri = __builtin_amdgcn_rsqf(fmaf(0.0f, 0.0f, fmaf(0.0f, 0.0f, fmaf(0.0f, 0.0f, e2f))));
                return (double)((float)J.m[iu] * ri);
            } else {
                const double r2 = fma(0.0, 0.0, fma(0.0, 0.0, fma(0.0, 0.0, eps2)));
                return J.m[iu] * (MIXED ? rinv_mixed(r2) : rinv_f64(r2));
            }
        };
        if constexpr (LPI >= 32 && AHEAD) {
            const LaneSums<LPI> sums(Q);
            if (!valid[u] || (lane & 15) != 0)
                continue;
#pragma unroll
            for (int n = 0; n < LaneSums<LPI>::N; ++n) {
                const int q = LaneSums<LPI>::quantity(n, js >> 4);
                double v = sums.v[n];
                if (q == NV)
                    v += self_phi();
                if (q < 0 || (q == NV && !PHI))
                    continue;
                if (part)
                    put<COH>(part + ((int64_t)b * 10 + q) * n_act_total + ku, v);
                else if (q < NV)
                    (q < 3 ? out.vec[0] : (q < 6 ? out.vec[1] : out.vec[2]))[ku * out.sk + (q % 3) * out.sd] = v;
                else if (out.pot)
                    out.pot[ku] = v;
            }
            continue;
        }
#pragma unroll
        for (int q = 0; q < NV + 1; ++q)
            Q[q] = lane_sum<LPI>(Q[q]);
        if (!valid[u] || js != 0)
            continue;
        Q[NV] += self_phi();
        if (part) {
            double *pb = part + (int64_t)b * 10 * n_act_total + ku;
#pragma unroll
            for (int q = 0; q < 10; ++q)
                put<COH>(pb + (int64_t)q * n_act_total, Q[q]);
        } else {
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int d = 0; d < 3; ++d)
                    out.vec[q][ku * out.sk + d * out.sd] = Q[3 * q + d];
            if (out.pot)
                out.pot[ku] = Q[NV];
        }
    }
}

}  // namespace

}  // namespace nb
