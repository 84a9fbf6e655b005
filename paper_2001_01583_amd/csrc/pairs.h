// Real-space Ewald pairs (Eq. (11)) on one wavefront, shared by the cell-list
// sum (k_ewald.hip) and the direct sum (k_misc.hip).
//
// A wavefront takes one ion at a time and 64 candidate partners at once.
// Only a sixth of the partners that cells or the whole box offer lie within
// the cut-off, and a pair's energy and force cost about ten times its
// distance test, so the accepted partners are queued in LDS and evaluated 64
// at a time with every lane at work.  (One ion per lane, each evaluating its
// partner as it is found, executed the pair terms for nearly every
// candidate, because some lane of 64 nearly always accepts.)  The order of
// the sums is fixed by the order of the candidates.
#pragma once

#include <hip/hip_runtime.h>

#include "wave_reduce.h"

namespace hpnfft {

// exp(x^2) erfc(x) for x >= 0 as G(t) / (x + 2), t = (x - 2) / (x + 2): G is
// smooth on the whole half-line (the mapping of Shepherd and Laframboise,
// Math. Comp. 36 (1981) 249); its Chebyshev interpolant of degree 26, in
// monomials, is within 4e-16 (relative) of the function.
__device__ inline double erfcx_pos(double x)
{
    constexpr double c[27] = {
    1.021582705242023, -0.6871606844138102, 0.2794720925560547,
    -0.036442231506922836, -0.021510661889486426, 0.006479185069310028,
    0.003090612059312434, -0.0008372960886356153, -0.000663073509073882,
    3.4371680319347264e-05, 0.00014447079620046643, 3.414748054725252e-05,
    -2.1696532340109436e-05, -1.611548837469618e-05, -1.1244034778588728e-06,
    3.629500461679375e-06, 1.999362119581824e-06, 2.8346296513609118e-08,
    -5.676806673916438e-07, -3.581655803025121e-07, -6.5759272455207115e-09,
    1.3983198251622205e-07, 5.99915938182997e-08, -2.661965682341084e-08,
    -2.0155627393974865e-08, 2.1479412981215555e-09, 2.5131744537192395e-09};
    const double y = x + 2.0;
    double r = __builtin_amdgcn_rcp(y);
    r = fma(fma(-y, r, 1.0), r, r);
    r = fma(fma(-y, r, 1.0), r, r);
    const double t = (x - 2.0) * r, t2 = t * t;
    double ev = c[26], od = c[25];
#pragma unroll
    for (int k = 24; k >= 0; k -= 2) ev = fma(ev, t2, c[k]);
#pragma unroll
    for (int k = 23; k >= 1; k -= 2) od = fma(od, t2, c[k]);
    return fma(t, od, ev) * r;
}

// Partial sums of one ion: energy (of its own pairs, halved) and force.
struct PairSum {
    double e, fx, fy, fz;
};
// Pair with separation (dx, dy, dz), squared distance d2 and charge product
// qq: erfc and the force's Gaussian share one exponential, the divisions are
// by one reciprocal square root.
__device__ inline void add_pair(double dx, double dy, double dz, double d2, double qq, double alpha, double c2,
                                PairSum &s)
{
    const double rinv = rsqrt(d2);
    const double d = d2 > 0.0 ? d2 * rinv : 0.0;  // (coincident ions: infinite energy)
    const double x = alpha * d;
    const double ex = exp(-x * x);
    const double ec = ex * erfcx_pos(x) * rinv;
    s.e += 0.5 * qq * ec;
    const double g = qq * fma(c2, ex, ec) * (rinv * rinv);
    s.fx = fma(g, dx, s.fx);
    s.fy = fma(g, dy, s.fy);
    s.fz = fma(g, dz, s.fz);
}

// Candidates in LDS (structure of arrays) and a wavefront's queue of accepted
// ones (a ring of 128 slots: at most 63 wait when 64 more are tested).
constexpr int kPairCap = 4096;
template <int CAP> struct PairTileOf {
    double x[CAP], y[CAP], z[CAP], q[CAP];
};
using PairTile = PairTileOf<kPairCap>;
constexpr int kPairQueue = 128;

// All pairs of the ion p (x, y, z, charge) with candidates 0 .. cnt - 1
// closer than rcut, except candidate `self`.  IMAGE: take each candidate's
// nearest periodic image (else the tile already holds it).
template <bool IMAGE, typename Tile>
__device__ inline void sweep_pairs(const double4 p, int self, int cnt, const Tile &t, unsigned short *queue,
                                   double rcut2, double alpha, double c2, double L, double invL, PairSum &s)
{
    const int lane = threadIdx.x & 63;
    int head = 0, n = 0;  // queue: first slot and length
    auto sep = [&](int k, double &dx, double &dy, double &dz) __attribute__((always_inline)) {
        dx = p.x - t.x[k];
        dy = p.y - t.y[k];
        dz = p.z - t.z[k];
        if (IMAGE) {
            dx -= L * rint(dx * invL);
            dy -= L * rint(dy * invL);
            dz -= L * rint(dz * invL);
        }
        return dx * dx + dy * dy + dz * dz;
    };
    auto evaluate = [&](int m) __attribute__((always_inline)) {
        // (the queue entries were written by other lanes of this wavefront:
        // LDS operations of a wavefront complete in order)
        __builtin_amdgcn_wave_barrier();
        if (lane < m) {
            const int k = queue[(head + lane) & (kPairQueue - 1)];
            double dx, dy, dz;
            const double d2 = sep(k, dx, dy, dz);
            add_pair(dx, dy, dz, d2, p.w * t.q[k], alpha, c2, s);
        }
        head += m;
        n -= m;
    };
    for (int k0 = 0; k0 < cnt; k0 += 64) {
        const int k = k0 + lane;
        bool in = false;
        if (k < cnt && k != self) {
            double dx, dy, dz;
            in = !(sep(k, dx, dy, dz) >= rcut2);  // (a NaN separation is accepted, and reaches the sums)
        }
        const unsigned long long mask = __ballot(in);
        if (in) {
            const int o = __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
            queue[(head + n + o) & (kPairQueue - 1)] = (unsigned short)k;
        }
        n += __popcll(mask);
        if (n >= 64) evaluate(64);
    }
    if (n > 0) evaluate(n);
}

// Force of an ion from its wavefront's partial sums: component c in the
// first lane of 16-lane row {0, 2, 1}[c].
__device__ inline double force_sum(const PairSum &s)
{
    double v = halve16(halve32(s.fx, s.fy), halve32(s.fz, 0.0));
    v += dpp<0x128>(v);  // row_ror:8
    return sum8(v);
}
// Adds the force to out[3] (or stores it) from the lanes that hold it.
__device__ inline void store_force(const PairSum &s, double *out, bool add)
{
    const double v = force_sum(s);
    const int lane = threadIdx.x & 63, row = lane >> 4;
    if ((lane & 15) == 0 && row < 3) {
        const int c = row == 0 ? 0 : (row == 1 ? 2 : 1);
        out[c] = add ? out[c] + v : v;
    }
}

// Sum of one value per thread over the workgroup in a fixed order (red: one
// double per wavefront); the result is valid in thread 0.
__device__ inline double block_sum_fixed(double v, double *red)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
    return t;
}

}  // namespace hpnfft
