// Start-up evaluation of nbody_init on gfx950: acceleration and jerk of every
// particle from positions and velocities (pass 1), then snap and crackle from
// those (pass 2), both in FP64 from the stored state whatever the precision.
//
// Bound: FP64 vector issue (a wave's FP64 instruction takes ~4.4 cycles at a
// clock of ~2.13 GHz under this load, measured), so the count of operations
// per pair is what matters.  Each pass forms only what it returns; with d, v,
// a, j the differences of position, velocity, acceleration and jerk,
// rho = 1 / r^2, w = m / r^3, alpha = (d.v) rho, beta = (v.v + d.a) rho +
// alpha^2, gamma = (3 v.a + d.j) rho + alpha (3 beta - 4 alpha^2),
//   p = v - 3 alpha d                           a  = sum w d, da = sum w p
//   s = a - 6 alpha p - 3 beta d                d2a = sum w s
//   c = j - 9 alpha s - 9 beta p - 3 gamma d    d3a = sum w c
// Every term is completed within its pair, where its parts largely cancel.
// (The parts summed apart over all pairs, with the factors 3, 6, 9 applied to
// the sums, take 72 operations instead of 76 in pass 2, 10.3 instead of 10.6
// ms at 65,536 bodies, but the rms error of the jerk at 4096 bodies over 30
// spheres was 6.1e-16 with them and one chain of split sums, and is 5.2e-16.)
// 31 FP64 operations per pair in pass 1 and 76 in pass 2.  Measured at 65,536
// bodies: pass 1 4.64 ms (926 G pairs/s), pass 2 10.6 ms (405 G pairs/s);
// one kernel with all four terms took 14.3 ms in either pass.
// Two particles per lane, so that each source's LDS reads serve two pairs (with
// the parts summed apart: 4.68 and 10.3 ms, with one per lane 5.02 and 10.8).
#include "force_body.h"

namespace nb {

namespace {

constexpr int SU_NT = 256;   // sources per LDS tile = lanes per workgroup

// One source in LDS.  16-byte multiples whose word stride keeps neighbouring
// lanes' 128-bit reads on different banks (20 and 28 words).
template <int PASS>
struct alignas(16) SuSrc {
    double x, y, z, m, vx, vy, vz, pad[3];
};
template <>
struct alignas(16) SuSrc<2> {
    double x, y, z, m, vx, vy, vz, ax, ay, az, jx, jy, jz, pad;
};

// LPI lanes per particle, IPT particles per lane group; a workgroup takes
// i-block blockIdx.x of its cluster against source split blockIdx.y.  Sums
// go to out0 / out1 (components [3][n]) or, with part != nullptr, to
// part[(b 6 + q) n + i].
template <int PASS, int LPI, int IPT, bool EPS0>
__global__ __launch_bounds__(SU_NT) void startup_kernel(State st, int64_t n, ForceWork w,
                                                        double *out0, double *out1, double *part,
                                                        double eps2)
{
    constexpr int GI = SU_NT / LPI;        // lane groups per workgroup
    constexpr int IB = GI * IPT;           // particles per workgroup
    __shared__ SuSrc<PASS> tl[SU_NT];
    const int64_t g = blockIdx.x;
    const int b = blockIdx.y;
    int64_t o0 = 0, o1 = n, gfirst = 0;
    if (w.blk_cluster) {
        const int c = w.blk_cluster[g];
        if (c < 0)
            return;   // grid padding past the last i-block
        gfirst = w.blk_first[c];
        o0 = w.off[c];
        o1 = w.off[c + 1];
    }
    const int64_t used = splits_used(o1 - o0, w.split, SU_NT);
    if (b >= used)
        return;       // no sources left for this split
    const int64_t j0 = o0 + split_begin(o1 - o0, used, SU_NT, b);
    const int64_t j1 = o0 + split_begin(o1 - o0, used, SU_NT, b + 1);
    const double *X = st.pos, *Y = X + n, *Z = Y + n, *VX = st.vel, *VY = VX + n, *VZ = VY + n;
    const double *AX = st.acc, *AY = AX + n, *AZ = AY + n, *JX = st.jrk, *JY = JX + n,
                 *JZ = JY + n;

    const int tid = threadIdx.x, il = tid / LPI, js = tid % LPI;
    int64_t i[IPT];
    double xi[IPT], yi[IPT], zi[IPT], vxi[IPT], vyi[IPT], vzi[IPT];
    double axi[IPT], ayi[IPT], azi[IPT], jxi[IPT], jyi[IPT], jzi[IPT];
    double S[IPT][6];
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
        i[u] = o0 + (g - gfirst) * IB + il + u * GI;
        const int64_t k = i[u] < o1 ? i[u] : o0;
        xi[u] = X[k]; yi[u] = Y[k]; zi[u] = Z[k];
        vxi[u] = VX[k]; vyi[u] = VY[k]; vzi[u] = VZ[k];
        if constexpr (PASS == 2) {
            axi[u] = AX[k]; ayi[u] = AY[k]; azi[u] = AZ[k];
            jxi[u] = JX[k]; jyi[u] = JY[k]; jzi[u] = JZ[k];
        }
#pragma unroll
        for (int q = 0; q < 6; ++q)
            S[u][q] = 0.0;
    }

    for (int64_t t0 = j0; t0 < j1; t0 += SU_NT) {
        __syncthreads();
        const int64_t jj = t0 + tid;
        SuSrc<PASS> &d = tl[tid];
        if (jj < j1) {
            d.x = X[jj]; d.y = Y[jj]; d.z = Z[jj]; d.m = st.mass[jj];
            d.vx = VX[jj]; d.vy = VY[jj]; d.vz = VZ[jj];
            if constexpr (PASS == 2) {
                d.ax = AX[jj]; d.ay = AY[jj]; d.az = AZ[jj];
                d.jx = JX[jj]; d.jy = JY[jj]; d.jz = JZ[jj];
            }
        } else {
            d.x = NULL_POS; d.y = NULL_POS; d.z = NULL_POS; d.m = 0.0;
            d.vx = 0.0; d.vy = 0.0; d.vz = 0.0;
            if constexpr (PASS == 2) {
                d.ax = 0.0; d.ay = 0.0; d.az = 0.0;
                d.jx = 0.0; d.jy = 0.0; d.jz = 0.0;
            }
        }
        __syncthreads();
#pragma unroll 2
        for (int t = js; t < SU_NT; t += LPI) {
            const SuSrc<PASS> &s = tl[t];
#pragma unroll
            for (int u = 0; u < IPT; ++u) {
                const double dx = s.x - xi[u], dy = s.y - yi[u], dz = s.z - zi[u];
                const double r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2)));
                double rinv = rinv_f64(r2);
                if constexpr (EPS0)
                    rinv = r2 > 0.0 ? rinv : 0.0;
                const double rho = rinv * rinv, wt = s.m * rinv * rho;
                const double vx = s.vx - vxi[u], vy = s.vy - vyi[u], vz = s.vz - vzi[u];
                const double al = fma(dx, vx, fma(dy, vy, dz * vz)) * rho;
                const double a3 = -3.0 * al;
                const double px = fma(a3, dx, vx), py = fma(a3, dy, vy), pz = fma(a3, dz, vz);
                double *Q = S[u];
                if constexpr (PASS == 1) {
                    Q[0] = fma(wt, dx, Q[0]); Q[1] = fma(wt, dy, Q[1]); Q[2] = fma(wt, dz, Q[2]);
                    Q[3] = fma(wt, px, Q[3]); Q[4] = fma(wt, py, Q[4]); Q[5] = fma(wt, pz, Q[5]);
                } else {
                    const double ax = s.ax - axi[u], ay = s.ay - ayi[u], az = s.az - azi[u];
                    const double jx = s.jx - jxi[u], jy = s.jy - jyi[u], jz = s.jz - jzi[u];
                    const double vv = fma(vx, vx, fma(vy, vy, fma(vz, vz,
                                      fma(dx, ax, fma(dy, ay, dz * az)))));
                    const double va = fma(vx, ax, fma(vy, ay, vz * az));
                    const double tt = fma(3.0, va, fma(dx, jx, fma(dy, jy, dz * jz)));
                    const double aa = al * al;
                    const double b3 = -3.0 * fma(vv, rho, aa);
                    const double g3 = fma(a3, fma(-4.0, aa, -b3), -3.0 * (tt * rho));
                    const double a6 = a3 + a3, a9 = 3.0 * a3, b9 = 3.0 * b3;
                    const double sx = fma(a6, px, fma(b3, dx, ax)), sy = fma(a6, py, fma(b3, dy, ay)),
                                 sz = fma(a6, pz, fma(b3, dz, az));
                    Q[0] = fma(wt, sx, Q[0]); Q[1] = fma(wt, sy, Q[1]); Q[2] = fma(wt, sz, Q[2]);
                    Q[3] = fma(wt, fma(a9, sx, fma(b9, px, fma(g3, dx, jx))), Q[3]);
                    Q[4] = fma(wt, fma(a9, sy, fma(b9, py, fma(g3, dy, jy))), Q[4]);
                    Q[5] = fma(wt, fma(a9, sz, fma(b9, pz, fma(g3, dz, jz))), Q[5]);
                }
            }
        }
    }

#pragma unroll
    for (int u = 0; u < IPT; ++u) {
        double *R = S[u];
        // lanes of a particle, in a fixed order (xor butterfly)
#pragma unroll
        for (int msk = 1; msk < LPI; msk <<= 1)
#pragma unroll
            for (int q = 0; q < 6; ++q)
                R[q] += __shfl_xor(R[q], msk, 64);
        if (i[u] >= o1 || js != 0)
            continue;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            if (part)
                part[((int64_t)b * 6 + q) * n + i[u]] = R[q];
            else
                (q < 3 ? out0 : out1)[(q % 3) * n + i[u]] = R[q];
        }
    }
}

// sums over the splits in use, in a fixed order: every fourth split, then the
// four sums (one chain over 16 splits gave the acceleration at 4096 bodies an
// rms error of 1.56e-16, this 1.26e-16, 64 lanes' sums in a tree 1.27e-16; the
// same time, 3.8 us); one lane per (component, particle)
__global__ __launch_bounds__(256) void startup_reduce(const double *part, int32_t B, int64_t n,
                                                      const int64_t *off,
                                                      const int32_t *cluster_of, double *out0,
                                                      double *out1)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= 6 * n)
        return;
    const int q = (int)(t / n);
    const int64_t i = t - (int64_t)q * n;
    const int c = cluster_of ? cluster_of[i] : 0;
    const int64_t used = splits_used(cluster_of ? off[c + 1] - off[c] : n, B, SU_NT);
    double r[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
    for (int64_t b = 0; b < used; b += 4)
#pragma unroll
        for (int k = 0; k < 4; ++k)
            r[k] += b + k < used ? part[((b + k) * 6 + q) * n + i] : 0.0;
    (q < 3 ? out0 : out1)[(q % 3) * n + i] = (r[0] + r[1]) + (r[2] + r[3]);
}

using KStart = void (*)(State, int64_t, ForceWork, double *, double *, double *, double);

template <int PASS, bool EPS0>
KStart pick_startup(int lpi)
{
    switch (lpi) {
    case 1: return startup_kernel<PASS, 1, 2, EPS0>;
    case 4: return startup_kernel<PASS, 4, 1, EPS0>;
    case 16: return startup_kernel<PASS, 16, 1, EPS0>;
    default: return startup_kernel<PASS, 64, 1, EPS0>;
    }
}

}  // namespace

// Launch shape: the fewest lanes per particle (1 with two particles per
// lane, 4, 16, 64) with which the units of a workgroup and a tile of its
// cluster's sources still give the chip's 256 compute units four each, then
// splits of whole tiles up to eight workgroups per unit, while the 6 B n
// partial sums fit the split buffer.  Fewer lanes mean fewer LDS reads and no
// lane sums; more than eight workgroups per unit only add partial sums.  With
// clusters, one lane per particle only if at most an eighth of the pair slots
// is empty for want of a second particle, and the workgroups of all are counted
// as if their units were of the largest cluster's length, so that its walks
// are short against a compute unit's share of the whole.
StartupShape startup_shape(const Ctx &c)
{
    const int64_t want = 1024, most = 2048, n = c.n;
    const int64_t tiles = (c.sizes.largest + SU_NT - 1) / SU_NT;
    StartupShape s;
    int64_t units = 0;
    for (int lpi : {1, 4, 16, 64}) {
        s.lpi = lpi;
        s.ib = SU_NT / lpi * (lpi == 1 ? 2 : 1);
        s.n_blocks = c.nc == 1 ? (n + s.ib - 1) / s.ib : n / s.ib + c.nc + 1;
        int64_t slots = 0, slots1 = 0;
        units = 0;
        for (size_t k = 0; k + 1 < c.off.size(); ++k) {
            const int64_t nk = c.off[k + 1] - c.off[k], t = (nk + SU_NT - 1) / SU_NT;
            units += (nk + s.ib - 1) / s.ib * t;
            slots += (nk + s.ib - 1) / s.ib * s.ib * t;
            slots1 += t * SU_NT * t;
        }
        if (units >= want && (c.nc == 1 || lpi > 1 || slots <= slots1 + slots1 / 8))
            break;
    }
    s.split = 1;
    while (units * s.split * 2 <= most * tiles && s.split * 2 <= tiles &&
           (int64_t)s.split * 2 * 6 * n <= 10 * c.part_cap)
        s.split *= 2;
    return s;
}

hipError_t launch_startup(Ctx &c, const ForceWork &w, const StartupShape &sh, int pass,
                          hipStream_t s)
{
    double *o0 = pass == 1 ? c.st.acc : c.st.snp, *o1 = pass == 1 ? c.st.jrk : c.st.crk;
    double *part = sh.split > 1 ? c.part : nullptr;
    const bool e0 = c.eps == 0.0;
    KStart k = pass == 1 ? (e0 ? pick_startup<1, true>(sh.lpi) : pick_startup<1, false>(sh.lpi))
                         : (e0 ? pick_startup<2, true>(sh.lpi) : pick_startup<2, false>(sh.lpi));
    hipLaunchKernelGGL(k, dim3((unsigned)sh.n_blocks, (unsigned)sh.split), dim3(SU_NT), 0, s, c.st,
                       c.n, w, o0, o1, part, c.eps * c.eps);
    if (part)
        hipLaunchKernelGGL(startup_reduce, dim3((unsigned)((6 * c.n + 255) / 256)), dim3(256), 0,
                           s, (const double *)part, sh.split, c.n, (const int64_t *)c.d_off,
                           (const int32_t *)(c.nc > 1 ? c.d_cluster_of : nullptr), o0, o1);
    return hipGetLastError();
}

}  // namespace nb
