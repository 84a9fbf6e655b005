// Interpolation by gathering (the Interpolating step of Algorithm 5): one
// wavefront per point reads the point's window from the grid and sums it.
//
// Every point is evaluated once, by one wavefront, in a fixed order, and its
// outputs are stored once: no LDS tile, no halo, no partial sums to add up,
// no clearing.  The price is that nothing is shared between points: (2m)^3
// complex values per point come from the caches.  Lane <-> (dim 1, dim 2) tap
// row of the window (64 rows at a time); a row's 2m values along dim 0 load
// back to back, so that a wavefront has 2m loads of 64 rows in flight.  The
// values every lane shares (header, dim-0 weights) come through scalar loads.
//
// Points are sorted by bin (or by line), so neighbouring points read
// neighbouring cells; workgroups are dealt to the eight XCDs round robin, so
// workgroup b takes the points of one of eight contiguous shares of the
// sorted points, and an XCD's L2 serves one region of the grid.
//
// Bound by the caches' read rate and latency: 64 KB per point (float64, 2m =
// 16) arrive at 17 TB/s.  Measured, with gradients: 165,888 ions on a 256^3
// grid 1.11 -> 0.64 ms (float64, 2m = 16) and 0.32 -> 0.18 ms (float32, 2m =
// 8) against boxes of the grid in LDS that every point's window meets about
// eight of; 200,000 points on 96^3, 1.54 -> 0.56 ms (2m = 16), 1.01 -> 0.33 ms
// (2m = 12) and 0.130 -> 0.077 ms (float32, 2m = 8) against the staged line
// sweep.  Without gradients the line sweeps stay faster on dense sets (N =
// 64^3, M = 2^20: 2m = 16 1.29 against 2.66 ms, float32 2m = 8 0.10 against
// 0.36 ms).  64 or 128 threads per workgroup: 3 to 5% slower.
#include <algorithm>

#include "internal.h"
#include "wave_reduce.h"

namespace hpnfft {

constexpr int kGatherThreads = 256;

template <typename R> struct Complex;
template <> struct Complex<float> { typedef float T __attribute__((ext_vector_type(2))); };
template <> struct Complex<double> { typedef double T __attribute__((ext_vector_type(2))); };

// which: every point of the plan, or those of the transforms that use boxes
// (Xform::goff: points of such transforms before this one).
//
// SPLIT (float32 gradients, 2m = 8): a line record's window is summed in the
// parts that the slabs of Zs planes cut it into, each part over the lanes
// first, and column slots stay on their lanes: the order in which the staged
// line sweeps add, so that the sums of a given grid (which the differentiable
// transform and the Ewald forces return widened to float64) are theirs bit for bit.
// Bound by the compute unit's scalar unit; its own branch with 32-bit element
// indices, all weights loaded at once and no conditions where no slab cuts the
// window: N = 64^3, 2^20 points 0.62 -> 0.39 ms, 2^21 points 1.24 -> 0.78 ms (the
// staged line sweep: 0.47 and 0.85 ms).
// A box record's window likewise (Zs > 0), in the parts that the boxes of gbox
// bins cut it into, the rows of a part on consecutive lanes (165,888 ions on
// 256^3: 0.18 ms, 0.09 ms as one sum per window, which moves the Ewald forces by
// 2.8e-7).
template <typename R, int M2, bool GRAD>
__global__ __launch_bounds__(kGatherThreads) void k_interp_gather(const Xform *__restrict__ xfs, int B, int which, int Zs,
                                                                  int zinv, long long total, long long per_xcd,
                                                                  const unsigned char *__restrict__ rec,
                                                                  int rec_bytes, R *__restrict__ outs)
{
    constexpr int m = M2 / 2, NO = GRAD ? 4 : 1, ROWS = M2 * M2;
    constexpr int OFF_PZ = (int)rec_off_pz(M2, sizeof(R));
    constexpr int OFF_D = (int)rec_prefix(M2, sizeof(R)) / (int)sizeof(R);
    constexpr bool SPLIT = GRAD && sizeof(R) == 4 && M2 == 8;
    using C = typename Complex<R>::T;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // this workgroup's points: share (index mod 8), in order
    const long long group = group_index();
    const long long k = group / kXcds * (kGatherThreads / 64) + wave;
    const long long g = group % kXcds * per_xcd + k;
    if (k >= per_xcd || g >= total) return;
    // the transform of point g: the last whose first point is not past it
    auto first = [&](const Xform *X) __attribute__((always_inline)) {
        return which == GATHER_ALL ? X->poff : X->goff;
    };
    int lo = 0, hi = B;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (first(xfs + mid) <= g) lo = mid;
        else hi = mid;
    }
    const Xform *X = xfs + lo;
    const long long pos = X->poff + (g - first(X));
    const int n0 = X->n[0], n1 = X->n[1], n2 = X->n[2];
    const unsigned char *rp = rec + (size_t)pos * rec_bytes;
    const cptr<int> hd = as_const(reinterpret_cast<const int *>(rp + OFF_PZ));
    const PointHead h = unpack_head(hd[0], hd[1], X->nbox[0] > 0);
    const cptr<R> pc = as_const(reinterpret_cast<const R *>(rp));
    const R *ps = reinterpret_cast<const R *>(rp);
    // dim 0: the slot order of the line records holds plane q in slot q mod
    // 2m, the box records are in tap order.  Either way slot s is tap (s -
    // rot) mod 2m.
    const int f0 = h.c0 - m + 1;
    int rot = 0;
    if (h.lines) {
        rot = f0 % M2;
        rot += rot < 0 ? M2 : 0;
    }
    // dim 2 of blocked line records: tap t in slot (t + line) mod 2m
    const int xr = h.xr;
    R v[2 * NO];
#pragma unroll
    for (int q = 0; q < 2 * NO; ++q) v[q] = R(0);
    const gptr<const C> grid = as_global(reinterpret_cast<const C *>(X->grid));
    const size_t pstride = (size_t)n1 * n2;
    if constexpr (SPLIT) {
        // dim-0 weights and derivatives: loaded within the parts' conditions, each
        // would be waited for by itself
        R w0[M2], e0[M2];
#pragma unroll
        for (int s = 0; s < M2; ++s) {
            w0[s] = pc[s];
            e0[s] = pc[OFF_D + s];
        }
        if (h.lines) {
            const int t1 = lane >> 3, s2 = lane & 7, t2 = (s2 - xr) & 7;
            int l1 = h.c1 - m + 1 + t1, l2 = h.c2 - m + 1 + t2;
            l1 += l1 < 0 ? n1 : (l1 >= n1 ? -n1 : 0);
            l2 += l2 < 0 ? n2 : (l2 >= n2 ? -n2 : 0);
            // (element indices stay below 2^30, so the scalar unit, which most of
            // this runs on, multiplies 32 bits)
            const gptr<const C> row = grid + (unsigned)(l1 * n2 + l2);
            const unsigned ps32 = (unsigned)pstride;
            const R w1 = ps[M2 + t1], w2 = ps[2 * M2 + s2], e1 = ps[OFF_D + M2 + t1], e2 = ps[OFF_D + 2 * M2 + s2];
            C c[M2];
            const bool inside = f0 >= 0 && f0 + M2 <= n0;
            if (inside) {
#pragma unroll
                for (int s = 0; s < M2; ++s) c[s] = row[(unsigned)(f0 + ((s - f0) & 7)) * ps32];
            } else {
#pragma unroll
                for (int s = 0; s < M2; ++s) {
                    int l0 = f0 + ((s - f0) & 7);
                    l0 += l0 < 0 ? n0 : (l0 >= n0 ? -n0 : 0);
                    c[s] = row[(unsigned)l0 * ps32];
                }
            }
            const R w12 = w1 * w2, d1 = e1 * w2, d2 = w1 * e2;
            auto part = [&](auto &&holds) __attribute__((always_inline)) {  // sum of the taps it holds
                R sr = R(0), si = R(0), dr = R(0), di = R(0);
#pragma unroll
                for (int s = 0; s < M2; ++s) {
                    if (!holds((s - f0) & 7)) continue;
                    sr = fma(w0[s], c[s][0], sr);
                    si = fma(w0[s], c[s][1], si);
                    dr = fma(e0[s], c[s][0], dr);
                    di = fma(e0[s], c[s][1], di);
                }
                const R a0 = halve32(sr * w12, si * w12), a1 = halve32(dr * w12, di * w12);
                const R a2 = halve32(sr * d1, si * d1), a3 = halve32(sr * d2, si * d2);
                return halve8_sum(halve16(a0, a1), halve16(a2, a3));
            };
            // the first slab edge at or after the first tap, as a tap (zinv =
            // 65536 / Zs + 1: exact for planes below 1024 and slabs of up to 64)
            auto slab_end = [&](int ta) __attribute__((always_inline)) {
                int l0 = f0 + ta;
                l0 += l0 < 0 ? n0 : (l0 >= n0 ? -n0 : 0);
                return min(M2, ta + min(n0, ((l0 * zinv >> 16) + 1) * Zs) - l0);
            };
            int tb = slab_end(0);  // taps up to tb - 1 end at a slab's edge, or at the wrap
            R total;
            if (tb == M2) {
                total = part([](int) { return true; });
            } else {
                total = R(0);
                for (int ta = 0; ta < M2; ta = tb) {
                    tb = slab_end(ta);
                    total += part([&](int t) { return t >= ta && t < tb; });
                }
            }
            if ((lane & 7) == 0) {
                const int j = lane >> 3;
                outs[pos * 8 + (((j & 1) << 2) | (j & 2) | (j >> 2))] = total;
            }
            return;
        }
        if (Zs > 0) {
            // taps that begin a box or the grid: lane 8 d + t <-> tap t of dim d
            const int d = lane >> 3;
            const int n = d == 0 ? n0 : d == 1 ? n1 : n2;
            const int nb = d == 0 ? X->nbox[0] : d == 1 ? X->nbox[1] : X->nbox[2];
            const int gb = d == 0 ? X->gbox[0] : d == 1 ? X->gbox[1] : X->gbox[2];
            int l = (d == 0 ? f0 : (d == 1 ? h.c1 : h.c2) - m + 1) + (lane & 7);
            l += l < 0 ? n : (l >= n ? -n : 0);
            const int bin = box_of(l, n, nb);
            const unsigned cuts = (unsigned)__ballot(bin % gb == 0 && box_lo(bin, n, nb) == l);
            auto next = [&](int d, int t) __attribute__((always_inline)) {  // (tap M2 ends the window)
                return __builtin_ctz((cuts >> (8 * d) & 0xfe | 0x100) >> (t + 1)) + t + 1;
            };
            R sum = R(0);
            for (int a1 = 0, b1; a1 < M2; a1 = b1) {
                b1 = next(1, a1);
                for (int a2 = 0, b2; a2 < M2; a2 = b2) {
                    b2 = next(2, a2);
                    const int w = b2 - a2;
                    const bool in = lane < (b1 - a1) * w;
                    // lane / w = lane inv >> 9
                    const int inv = __builtin_amdgcn_readfirstlane((int)(512.0f * __builtin_amdgcn_rcpf((float)w))) + 1;
                    const int r1 = in ? lane * inv >> 9 : 0, t1 = a1 + r1, t2 = a2 + (in ? lane - r1 * w : 0);
                    int l1 = h.c1 - m + 1 + t1, l2 = h.c2 - m + 1 + t2;
                    l1 += l1 < 0 ? n1 : (l1 >= n1 ? -n1 : 0);
                    l2 += l2 < 0 ? n2 : (l2 >= n2 ? -n2 : 0);
                    const gptr<const C> row = grid + ((size_t)l1 * n2 + l2);
                    const R w1 = ps[M2 + t1], w2 = ps[2 * M2 + t2];
                    const R e1 = ps[OFF_D + M2 + t1], e2 = ps[OFF_D + 2 * M2 + t2];
                    C c[M2];
                    if (in) {
#pragma unroll
                        for (int t = 0; t < M2; ++t) {
                            int l0 = f0 + t;
                            l0 += l0 < 0 ? n0 : (l0 >= n0 ? -n0 : 0);
                            c[t] = row[(size_t)l0 * pstride];
                        }
                    } else {
#pragma unroll
                        for (int t = 0; t < M2; ++t) c[t] = C{0, 0};
                    }
                    const R w12 = w1 * w2, d1 = e1 * w2, d2 = w1 * e2;
                    for (int a0 = 0, b0; a0 < M2; a0 = b0) {
                        b0 = next(0, a0);
                        R sr = R(0), si = R(0), dr = R(0), di = R(0);
#pragma unroll
                        for (int t = 0; t < M2; ++t) {
                            if (t < a0 || t >= b0) continue;
                            sr = fma(w0[t], c[t][0], sr);
                            si = fma(w0[t], c[t][1], si);
                            dr = fma(e0[t], c[t][0], dr);
                            di = fma(e0[t], c[t][1], di);
                        }
                        const R p0 = halve32(sr * w12, si * w12), p1 = halve32(dr * w12, di * w12);
                        const R p2 = halve32(sr * d1, si * d1), p3 = halve32(sr * d2, si * d2);
                        sum += halve8_sum(halve16(p0, p1), halve16(p2, p3));
                    }
                }
            }
            if ((lane & 7) == 0) {
                const int j = lane >> 3;
                outs[pos * 8 + (((j & 1) << 2) | (j & 2) | (j >> 2))] = sum;
            }
            return;
        }
    }
#pragma unroll 1
    for (int i = lane; i < ((ROWS + 63) / 64) * 64; i += 64) {
        const int ic = ROWS % 64 == 0 ? i : min(i, ROWS - 1);  // (lanes past the last row repeat it with weight 0)
        // (lane <-> column slot: tap t in slot (t + xr) mod 2m)
        const int t1 = ic / M2, s2 = ic - t1 * M2;
        const int t2 = s2 - xr + (s2 < xr ? M2 : 0);
        int l1 = h.c1 - m + 1 + t1, l2 = h.c2 - m + 1 + t2;
        l1 += l1 < 0 ? n1 : (l1 >= n1 ? -n1 : 0);
        l2 += l2 < 0 ? n2 : (l2 >= n2 ? -n2 : 0);
        const gptr<const C> row = grid + ((size_t)l1 * n2 + l2);
        const R w1 = ROWS % 64 == 0 || i < ROWS ? ps[M2 + t1] : R(0), w2 = ps[2 * M2 + s2];
        C c[M2];
#pragma unroll
        for (int s = 0; s < M2; ++s) {
            int t = s - rot;
            t += t < 0 ? M2 : 0;
            int l0 = f0 + t;
            l0 += l0 < 0 ? n0 : (l0 >= n0 ? -n0 : 0);
            c[s] = row[(size_t)l0 * pstride];
        }
        R sr = R(0), si = R(0), dr = R(0), di = R(0);
#pragma unroll
        for (int s = 0; s < M2; ++s) {
            const R w = pc[s];
            sr = fma(w, c[s][0], sr);
            si = fma(w, c[s][1], si);
            if constexpr (GRAD) {
                const R dw = pc[OFF_D + s];
                dr = fma(dw, c[s][0], dr);
                di = fma(dw, c[s][1], di);
            }
        }
        const R w12 = w1 * w2;
        v[0] = fma(sr, w12, v[0]);
        v[1] = fma(si, w12, v[1]);
        if constexpr (GRAD) {
            const R d1 = (ROWS % 64 == 0 || i < ROWS ? ps[OFF_D + M2 + t1] : R(0)) * w2, d2 = w1 * ps[OFF_D + 2 * M2 + s2];
            v[2] = fma(dr, w12, v[2]);
            v[3] = fma(di, w12, v[3]);
            v[4] = fma(sr, d1, v[4]);
            v[5] = fma(si, d1, v[5]);
            v[6] = fma(sr, d2, v[6]);
            v[7] = fma(si, d2, v[7]);
        }
    }
    if constexpr (GRAD) {
        // the eight sums through the halving steps of wave_reduce.h: the
        // 8-lane group j ends with the sum of value bitrev3(j)
        const R a0 = halve32(v[0], v[1]), a1 = halve32(v[2], v[3]);
        const R a2 = halve32(v[4], v[5]), a3 = halve32(v[6], v[7]);
        const R r = halve8_sum(halve16(a0, a1), halve16(a2, a3));
        if ((lane & 7) == 0) {
            const int j = lane >> 3;
            outs[pos * (2 * NO) + (((j & 1) << 2) | (j & 2) | (j >> 2))] = r;
        }
    } else {
        // each value fed in four times: lanes 0-31 end with the sum of v[0],
        // lanes 32-63 with that of v[1]
        const R a = halve32(v[0], v[1]);
        const R b = halve16(a, a);
        const R r = halve8_sum(b, b);
        if ((lane & 31) == 0) outs[pos * 2 + (lane >> 5)] = r;
    }
}

template <typename R, int M2>
static hipError_t gather_m(bool grad, const Xform *dxf, int B, int which, int Zs, long long total, const unsigned char *rec,
                           size_t rec_bytes, R *outs, hipStream_t s)
{
    constexpr int W = kGatherThreads / 64;
    const long long per_xcd = (total + kXcds - 1) / kXcds;
    const dim3 grid = launch_grid((per_xcd + W - 1) / W * kXcds, kGatherThreads);
    auto kern = grad ? k_interp_gather<R, M2, true> : k_interp_gather<R, M2, false>;
    hipLaunchKernelGGL(kern, grid, dim3(kGatherThreads), 0, s, dxf, B, which, Zs,
                       Zs > 0 ? 65536 / Zs + 1 : 0, total, per_xcd, rec,
                       (int)rec_bytes, outs);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_interp_gather(int m, bool grad, const Xform *dxf, int B, int which, int Zs, long long total,
                                const unsigned char *rec, size_t rec_bytes, R *outs, hipStream_t s)
{
    if (total <= 0) return hipSuccess;
    switch (m) {
#define HPNFFT_GATHER_CASE(MM) \
    case MM: return gather_m<R, 2 * MM>(grad, dxf, B, which, Zs, total, rec, rec_bytes, outs, s);
        HPNFFT_GATHER_CASE(1)
        HPNFFT_GATHER_CASE(2)
        HPNFFT_GATHER_CASE(3)
        HPNFFT_GATHER_CASE(4)
        HPNFFT_GATHER_CASE(5)
        HPNFFT_GATHER_CASE(6)
        HPNFFT_GATHER_CASE(7)
        HPNFFT_GATHER_CASE(8)
        HPNFFT_GATHER_CASE(9)
        HPNFFT_GATHER_CASE(10)
        HPNFFT_GATHER_CASE(11)
        HPNFFT_GATHER_CASE(12)
        HPNFFT_GATHER_CASE(13)
        HPNFFT_GATHER_CASE(14)
        HPNFFT_GATHER_CASE(15)
#undef HPNFFT_GATHER_CASE
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_interp_gather<double>(int, bool, const Xform *, int, int, int, long long,
                                                 const unsigned char *, size_t, double *, hipStream_t);
template hipError_t launch_interp_gather<float>(int, bool, const Xform *, int, int, int, long long,
                                                const unsigned char *, size_t, float *, hipStream_t);

}  // namespace hpnfft
