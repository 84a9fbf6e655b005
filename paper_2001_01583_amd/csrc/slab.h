// Slab spread for windows of 2m = 10 .. 16 cells (the Spreading step of
// Algorithm 2, Section 3) as matrix-core contractions.
//
// A work item is a tile of T x T z-lines restricted to a slab of Zs planes, as
// in the staged sweep (sweep.h).  A task is one line of the tile and four
// planes of the slab: the line's 2m x 2m footprint fits one 16 x 16 matrix,
// and the points of a line share it, so
//
//   D_q[y, x] += sum_p (f_p w1_p[y] w0_p[q]) w2_p[x]     (real, imaginary)
//
// takes four points per matrix instruction, plane and component, with no zero
// columns at 2m = 16.  A wavefront holds the four planes in accumulators,
// goes through the points whose windows reach them (2m + 3 planes of the
// line's sorted points, up to three runs with the periodic images) and adds
// the planes to the slab's tile in LDS once: 512 native LDS float64 adds per
// plane and line.  Float32 sums are added up in the tile in float64 too (the
// LDS float32 add is 13 times slower) and rounded once, and at most kSlabRun
// points of a line are added up in float32 before they join the tile: a crowded
// line's sums lost precision otherwise (400,000 points, half of them in 16
// clusters, N = 32^3, 2m = 14: error against 64 bits 7.0e-7 with whole lines,
// 3.2e-7 with runs of 64, 4.4e-7 for the staged sweep; both 0.33 ms).  Then all
// threads add the tile to the grid.
//
// Loads run one batch ahead, across tasks: the run bounds of the next task
// (six values, one per lane) are loaded while a task is worked off.
//
// Bound by the vector datapath, which executes the matrix instructions (64
// cycles for float64), then by the LDS adds.  Measured against the staged sweep
// it replaced for these windows (float64): N = 64^3, M = 2^20, 2m = 16 1.96 ->
// 0.82 ms, 2m = 12 1.36 -> 0.62 ms; 200,000 points on 96^3, 2m = 16 0.64 ->
// 0.24 ms; 150,001 points on 96 x 72 x 120, 2m = 12 0.45 -> 0.18 ms; 4096 points
// on 32^3 85 -> 28 us.
//
// Grids of one and two dimensions (flat): the window along the missing
// dimension is the cell 0 alone, so the plan has one slab and the sweep holds its
// first plane (d = 2, 256^2, 400,000 points, 2m = 16, float32 adjoint: 0.61 ms with
// all planes, 0.21 ms).
#pragma once

#include "mat.h"
#include "sweep.h"

namespace hpnfft {

constexpr int kSlabQuad = 4;  // planes per task
constexpr int kSlabRun = 64;  // points added up in float32 (a multiple of 4)
__host__ __device__ constexpr size_t slab_lds(int T, int Zs, int M2)
{
    return (size_t)Zs * (T + M2 - 1) * (T + M2 - 1) * 16;
}

// TT: the tile edge where it is known (0: T), for constant LDS strides.
template <typename R, int M2, int TT>
__global__ __launch_bounds__(1024) void k_spread_slab(const Xform *__restrict__ xfs, const SItem *__restrict__ items,
                                                      int nitems, int *__restrict__ queue, int T_, int Zs,
                                                      const unsigned char *__restrict__ rec, int rbytes,
                                                      const R *__restrict__ fs, const int *__restrict__ cell_start)
{
    static_assert(M2 <= 16 && block_w(M2) == 1, "one line's footprint per matrix");
    constexpr int m = M2 / 2, Q = kSlabQuad;
    constexpr int OFF_PZ = (int)rec_off_pz(M2, sizeof(R));
    using V4 = typename Mat<R>::V4;
    typedef R V2 __attribute__((ext_vector_type(2)));
    extern __shared__ uint4 smem16[];
    double *acc = reinterpret_cast<double *>(smem16);  // real parts [Zs][P][P], then imaginary parts
    __shared__ int s_item;
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wave = uni(tid >> 6), nw = nthr >> 6;
    const int p4 = lane >> 4, col = lane & 15;
    const int T = TT ? TT : T_, P = T + M2 - 1, plane = P * P, im = Zs * plane;
    const bool on = col < M2;
    const int cc = on ? col : 0;

    for (int i = tid; i < 2 * im; i += nthr) acc[i] = 0.0;  // the flushes leave the tile cleared
    for (int it = next_item(queue, &s_item); it < nitems; it = next_item(queue, &s_item)) {
        const SItem W = items[uni(it)];
        const Xform *X = xfs + W.xf;
        const int n0 = X->n[0], n1 = X->n[1], n2 = X->n[2], ntx = X->ntx;
        const int X0 = (W.tile % ntx) * T, Y0 = (W.tile / ntx) * T;
        const int z0 = W.slab * Zs, zs = min(Zs, n0 - z0);
        const long long poff = X->poff;
        const unsigned char *recb = rec + (size_t)poff * rbytes;
        const V2 *fsb = reinterpret_cast<const V2 *>(fs) + poff;
        const int *csb = cell_start + X->key_off + (long long)W.tile * T * T * n0;
        // tasks: line W.lb + t / nq, planes from z0 + Q (t % nq) on.  A
        // wavefront's line and quad advance by constant steps; lines / T by
        // multiplication (exact: fewer than 1024 lines, T <= 32).
        const bool flat = X->flat > 0;  // (plane 0 only receives anything)
        const int nq = flat ? 1 : (zs + Q - 1) / Q, nl = W.le - W.lb;
        const int dl = nw / nq, dq = nw - dl * nq;
        const int inv_t = 65536 / T + 1;
        // the dim-0 weights of four planes are one aligned vector when the
        // slots start at a multiple of four and do not depend on the image
        const bool vec = M2 % Q == 0 && z0 % Q == 0 && n0 % M2 == 0;

        // Sorted points of a task by periodic image u (shift u n0, u = -1, 0,
        // 1): those in grid planes c of [a - u n0, b - u n0], where a .. b =
        // z - m .. z + Q + m - 2 for the task's first plane z.  Lane 2 (u + 1)
        // loads the first point, lane 2 (u + 1) + 1 the end.
        auto bounds = [&](int l, int q) __attribute__((always_inline)) {
            int v = 0;
            if (l < nl && lane < 6) {
                const int z = z0 + Q * q;
                const int u = (lane >> 1) - 1;
                const int lo = max(z - m - u * n0, 0), hi = min(z + Q + m - 2 - u * n0, n0 - 1);
                if (lo <= hi) v = csb[(long long)(W.lb + l) * n0 + ((lane & 1) ? hi + 1 : lo)];
            }
            return v;
        };
        struct Runs {
            int p0, p1, p2, n0, n1, n;  // first points, lengths of the first two, points in all
        };
        auto unpack = [&](int v) __attribute__((always_inline)) {
            Runs r;
            r.p0 = __builtin_amdgcn_readlane(v, 0);
            r.p1 = __builtin_amdgcn_readlane(v, 2);
            r.p2 = __builtin_amdgcn_readlane(v, 4);
            r.n0 = __builtin_amdgcn_readlane(v, 1) - r.p0;
            r.n1 = __builtin_amdgcn_readlane(v, 3) - r.p1;
            r.n = r.n0 + r.n1 + __builtin_amdgcn_readlane(v, 5) - r.p2;
            return r;
        };
        // a lane's point of a batch: its value, weights and first tap plane
        // relative to the task's planes
        struct PointData {
            V2 f;
            V4 w0;
            R w1, w2;
            int c0, u;
        };
        auto fetch = [&](const Runs &r, int i, int z, PointData &d) __attribute__((always_inline)) {
            const int k = min(i + p4, r.n - 1);
            const bool b0 = k < r.n0, b1 = k < r.n0 + r.n1;
            const int sp = k + (b0 ? r.p0 : (b1 ? r.p1 - r.n0 : r.p2 - r.n0 - r.n1));
            d.u = b0 ? -n0 : (b1 ? 0 : n0);
            const unsigned char *rp = recb + (size_t)(unsigned)sp * (unsigned)rbytes;
            const R *ps = reinterpret_cast<const R *>(rp), *pcol = ps + cc;
            d.f = fsb[(unsigned)sp];
            d.w1 = pcol[M2];
            d.w2 = pcol[2 * M2];
            d.c0 = *reinterpret_cast<const int *>(rp + OFF_PZ);
            // slot of plane q: q mod 2m in the point's own frame
            if (vec) {
                d.w0 = *reinterpret_cast<const V4 *>(ps + (unsigned)z % M2);
            } else {
                int s = (z - d.u + M2) % M2;  // z - u n0 >= -M2 (windows reach no further)
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    d.w0[q] = ps[s];
                    ++s;
                    s = s == M2 ? 0 : s;
                }
            }
        };

        // the next task, its bounds (loaded one task ahead) and its first batch
        int line = wave / nq, quad = wave - line * nq;
        Runs r{};
        int bv = bounds(line, quad);
        PointData d;
        // from (line, quad) on, the first task that has points
        auto advance = [&](bool here) __attribute__((always_inline)) {
            for (;; here = false) {
                if (!here) {
                    line += dl;
                    quad += dq;
                    if (quad >= nq) {
                        quad -= nq;
                        ++line;
                    }
                }
                if (line >= nl) return;
                r = unpack(bv);
                const bool wrap = quad + dq >= nq;
                bv = bounds(line + dl + (wrap ? 1 : 0), quad + dq - (wrap ? nq : 0));
                if (r.n > 0) return;
            }
        };
        advance(true);
        if (line < nl) fetch(r, 0, z0 + Q * quad, d);
        while (line < nl) {
            const int z = z0 + Q * quad, li = W.lb + line;
            const int ly = (li * inv_t) >> 16, lx = li - ly * T;
            V4 re[Q], ie[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) re[q] = ie[q] = V4{0, 0, 0, 0};
            // the planes to the tile, and the accumulators cleared; the lane's
            // rows of a result: y0 + YS k
            constexpr int YS = sizeof(R) == 4 ? 1 : 4;
            const int y0 = sizeof(R) == 4 ? 4 * p4 : p4;
            double *cre = acc + (z - z0) * plane + (ly + y0) * P + lx + col, *cim = cre + im;
            auto flush = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    if (z + q < z0 + zs) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            if (on && y0 + YS * k < M2) {
                                atomicAdd(&cre[q * plane + YS * k * P], (double)re[q][k]);
                                atomicAdd(&cim[q * plane + YS * k * P], (double)ie[q][k]);
                            }
                        }
                    }
                    re[q] = ie[q] = V4{0, 0, 0, 0};
                }
            };
            const int n = r.n;
            int i = 0;
            do {
                const int end = sizeof(R) == 4 ? min(n, i + kSlabRun) : n;
                for (; i < end; i += 4) {
                    const int last = min(n - 1 - i, 3);
                    const int fr = d.c0 + d.u - (m - 1) - z;  // first tap plane
                    const int fmin = uni(fr), fmax = __builtin_amdgcn_readlane(fr, 16 * last);
                    const R w1 = on && p4 <= last ? d.w1 : R(0);
                    const R b = on ? d.w2 : R(0);
                    const R ar = d.f[0] * w1, ai = d.f[1] * w1;
                    R wr[Q], wi[Q];
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        const R w0 = (unsigned)(q - fr) < (unsigned)M2 ? d.w0[q] : R(0);
                        wr[q] = ar * w0;
                        wi[q] = ai * w0;
                    }
                    if (i + 4 < n) {
                        fetch(r, i + 4, z, d);
                    } else {
                        advance(false);
                        if (line < nl) fetch(r, 0, z0 + Q * quad, d);
                    }
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        // no point of the batch reaches the plane
                        if (q < fmin || q >= fmax + M2 || (q > 0 && flat)) continue;
                        re[q] = Mat<R>::mul(wr[q], b, re[q]);
                        ie[q] = Mat<R>::mul(wi[q], b, ie[q]);
                    }
                }
                flush();
            } while (i < n);
        }
        __syncthreads();
        // the tile to the grid; consecutive lanes add to consecutive reals
        const int ry0 = W.lb / T, nrows = (W.le - 1) / T + M2 - ry0;
        const gptr<R> grid = as_global(reinterpret_cast<R *>(X->grid));
        const int per = nrows * 2 * P;
        for (int i = tid; i < zs * per; i += nthr) {
            const int z = i / per, rem = i - z * per;
            const int y = ry0 + rem / (2 * P), xc = rem - (rem / (2 * P)) * 2 * P;
            const int x = xc >> 1, c = xc & 1;
            double *cell = acc + z * plane + y * P + x + c * im;
            const R v = (R)*cell;
            *cell = 0.0;
            if (v != R(0)) {
                const int gy = wrapn(Y0 + y - m + 1, n1), gx = wrapn(X0 + x - m + 1, n2);
                const size_t gi = (((size_t)(z0 + z) * n1 + gy) * n2 + gx) * 2 + c;
                __hip_atomic_fetch_add(&grid[gi], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        // (the next item begins with a barrier)
    }
    release_queue(queue);
}

template <typename R, int M2>
static hipError_t spread_slab(const Xform *dxf, const SItem *items, int nitems, int *queue, Tiling t,
                              const unsigned char *rec, size_t rec_bytes, const R *fs, const int *cs, hipStream_t s)
{
    const size_t lds = slab_lds(t.T, t.Zs, M2);
    auto kern = t.T == 8 ? k_spread_slab<R, M2, 8> : k_spread_slab<R, M2, 0>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    // as many workgroups per compute unit as the tiles leave room for, 1024
    // threads between them
    const int per_cu = std::max(1, std::min(4, (int)((160 * 1024) / (lds + 256))));
    const int threads = per_cu >= 4 ? 256 : (per_cu >= 2 ? 512 : 1024);
    const int grid = std::min(cu_count() * per_cu, nitems);
    if (grid < 1) return hipSuccess;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), lds, s, dxf, items, nitems, queue, t.T, t.Zs, rec,
                       (int)rec_bytes, fs, cs);
    return hipGetLastError();
}

}  // namespace hpnfft
