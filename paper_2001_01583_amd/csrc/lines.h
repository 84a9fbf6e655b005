// Interpolation by batches of points on a z-line, for windows of 2m = 10 ..
// 16 cells on line-method plans (the Interpolating step of Algorithm 5,
// Section 3), with or without the gradient.
//
// A work item is a group of 4 x 4 neighbouring z-lines and a range of their
// planes; the workgroup goes through it in phases of DZ planes, with the
// footprint of the points whose cells lie in a phase (DZ + 2m - 1 planes of
// (2m + 3)^2 cells) in an LDS ring.  Every point is evaluated once, in full,
// by one wavefront, and stored once.
//
// The points of a line share their tap rows and differ in their planes only,
// so a wavefront takes up to G consecutive points of a line together: it
// reads each plane of their windows' union from LDS once (lane <-> (dim 1,
// dim 2) tap rows, 64 at a time) and adds it to every point whose window
// holds it, with the dim-0 weight from a lane read.  At 0.5 points per cell
// four points of a line span 22 planes instead of 64.  The 2 G (with the
// gradient 8 per point) sums then go through the halving steps of
// wave_reduce.h together.
//
// Bound by the float64 vector unit (290 instructions per point at 2m = 16, 128
// of them the multiply-adds) at three or four wavefronts per SIMD.  Measured
// (float64) against what it replaced: N = 64^3, M = 2^20, 2m = 16 1.29 -> 0.99
// ms (groups of lines with register windows), 2m = 12 1.49 -> 0.65 ms (staged
// sweep); 150,001 points on 96 x 72 x 120, 2m = 12 0.40 -> 0.21 ms; float32, 2m =
// 16 0.89 -> 0.64 ms; with gradients, 200,000 points on 96^3, 2m = 16 0.47 ms
// against 0.56 for the gather.  Tried and slower: the next batch's records
// loaded while one is evaluated (2m = 16 1.31 ms), one plane per round (2m =
// 12 0.76 ms), three points per batch (as fast).
#pragma once

#include "sweep.h"

namespace hpnfft {

constexpr int kLineT = 4;  // lines per group along dims 1 and 2
// Planes per item at least, where whole phases would leave workgroups out: 32^3
// cells, 2m = 16, 200,000 points, float32 236 -> 134 us, float64 229 -> 160 us (three
// ranges of 13 planes before; register windows, 145 and 233 us).
constexpr int kLineZ = 4;

template <typename R, int M2, bool GRAD> struct LineBatch {
    static constexpr int P = kLineT + M2 - 1, PLANE = P * P;  // footprint cells of a plane
    static constexpr int G = GRAD ? 2 : 4;                    // points per batch
    static constexpr int RPG = 64 / M2;                       // tap rows per row group
    static constexpr int NR = (M2 + RPG - 1) / RPG;           // row groups
    // planes of new points per phase: a ring in half of the LDS (two
    // workgroups per compute unit) where that leaves at least 10, else in all
    // of it
    static constexpr int cells(size_t bytes) { return (int)(bytes / (PLANE * 2 * sizeof(R))); }
    static constexpr int half = cells(79 * 1024) - (M2 - 1), full = cells(158 * 1024) - (M2 - 1);
    static constexpr bool two = half >= 10 && !(sizeof(R) == 8 && M2 >= 12);
    static constexpr int DZ = two ? (half < 16 ? half : 16) : (full < 16 ? full : 16);
    static constexpr int NP = DZ + M2 - 1;  // ring planes
    // wavefronts per SIMD: the accumulators, two planes' rows and the next
    // phase's cells take more than 128 registers for wide float64 windows
    static constexpr int waves = sizeof(R) == 8 && M2 >= 14 ? 3 : 4;
    static constexpr int threads = (two ? 128 : 256) * waves;
    static constexpr size_t lds = (size_t)NP * PLANE * 2 * sizeof(R);
};

template <typename R, int M2, bool GRAD>
__global__ __launch_bounds__((LineBatch<R, M2, GRAD>::threads), (LineBatch<R, M2, GRAD>::waves)) void k_interp_lines(
    const Xform *__restrict__ xfs, int B, int ngroups, int ranges, int fine, int *__restrict__ queue, int T,
    const unsigned char *__restrict__ rec, int rbytes, const int *__restrict__ cell_start, R *__restrict__ outs)
{
    using LB = LineBatch<R, M2, GRAD>;
    constexpr int m = M2 / 2, G = LB::G, RPG = LB::RPG, NR = LB::NR, P = LB::P, PLANE = LB::PLANE, DZ = LB::DZ, NP = LB::NP;
    constexpr int NTH = LB::threads, NW = NTH / 64, NL = kLineT * kLineT;
    constexpr int NPF = (DZ * PLANE + NTH - 1) / NTH;
    constexpr int OFF_PZ = (int)rec_off_pz(M2, sizeof(R));
    constexpr int OFF_D = (int)rec_prefix(M2, sizeof(R)) / (int)sizeof(R);
    typedef R V2 __attribute__((ext_vector_type(2)));
    extern __shared__ uint4 smem16[];
    V2 *ring = reinterpret_cast<V2 *>(smem16);  // [plane mod NP][row][column]
    __shared__ int s_item;
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    // the lane's column t2 and tap rows t1 + RPG k; rows past the window and
    // the lanes left over read some cell of the footprint with weight 0
    const int t1 = lane / M2, t2 = lane - t1 * M2;
    const bool used = lane < RPG * M2;
    auto row_on = [&](int k) __attribute__((always_inline)) { return used && t1 + RPG * k < M2; };

    for (int it = next_item(queue, &s_item); it < ngroups * ranges; it = next_item(queue, &s_item)) {
        // item <-> (plane range, line group), neighbouring groups one after the
        // other.  (Read from LDS, the item's place stays in vector registers: as
        // scalars it made branches of the window tests, 2m = 16 0.96 -> 1.12 ms.)
        const int range_i = it / ngroups, gi = it - range_i * ngroups;
        const Xform *xf = xfs + xform_of(xfs, B, &Xform::lgoff, uni(gi));
        const int n0 = xf->n[0], n1 = xf->n[1], n2 = xf->n[2], ntx = xf->ntx;
        const int phases = (n0 + DZ - 1) / DZ, nr = min(fine ? (n0 + kLineZ - 1) / kLineZ : phases, ranges);
        const int Zi = fine ? (n0 + nr - 1) / nr : (phases + nr - 1) / nr * DZ;
        const int za = range_i * Zi, ze = min(za + Zi, n0);  // cells of the item's points
        if (za >= n0) continue;  // (a transform of fewer ranges)
        const int ngx = (n2 + kLineT - 1) / kLineT, gl = gi - xf->lgoff;
        const int X0 = (gl % ngx) * kLineT, Y0 = (gl / ngx) * kLineT;
        const long long poff = xf->poff;
        const unsigned char *recb = rec + (size_t)poff * rbytes;
        const gptr<const V2> grid = as_global(reinterpret_cast<const V2 *>(xf->grid));
        const size_t pstride = (size_t)n1 * n2;
        const int qb = za - m + 1;                              // its first window plane
        // a leading dim without a coordinate holds every point at plane 0, with
        // the unit impulse there: that plane only (ring numbering).  128
        // frequencies, 200,000 points, 2m = 16, float32 722 -> 251 us, float64 509 ->
        // 338 us (register windows: 314 and 392 us)
        const bool flat = xf->flat > 0;
        // sorted points of line `lane` (lanes 0 .. 15) in a phase's planes
        const int ly = (lane & 15) / kLineT, lx = lane & (kLineT - 1);
        const bool has = lane < NL && Y0 + ly < n1 && X0 + lx < n2;
        const int yl = min(Y0 + ly, n1 - 1), xl = min(X0 + lx, n2 - 1);
        const int q1 = yl / T, q2 = xl / T;
        const int *cs = cell_start + xf->key_off +
                        (long long)(((q1 * ntx + q2) * T + (yl - q1 * T)) * T + (xl - q2 * T)) * n0;
        int a0 = 0, a1 = 0;  // this phase's range, the next one's loaded ahead
        auto range = [&](int zc) __attribute__((always_inline)) {
            const bool ok = has && zc < ze;
            a0 = ok ? cs[zc] : 0;
            a1 = ok ? cs[min(zc + DZ, ze)] : 0;
        };
        // footprint cells of ring planes j0 .. j0 + nz - 1 (nz <= DZ), through registers
        V2 pf[NPF];
        auto planes_fetch = [&](int j0, int nz) __attribute__((always_inline)) {
            int t = tid;
            asm volatile("" : "+v"(t));  // (indices are cheaper computed per phase than kept in registers)
#pragma unroll
            for (int u = 0; u < NPF; ++u) {
                const int e = t + u * NTH;
                const int zz = e / PLANE, c = e - zz * PLANE;
                pf[u] = V2{0, 0};
                if (zz < nz) {
                    const int fy = c / P, fx = c - fy * P;
                    int gz = qb + j0 + zz, gy = Y0 + fy - (m - 1), gx2 = X0 + fx - (m - 1);
                    gz += gz < 0 ? n0 : 0;
                    gz -= gz >= n0 ? n0 : 0;
                    gz -= gz >= n0 ? n0 : 0;
                    gy += gy < 0 ? n1 : 0;
                    gy -= gy >= n1 ? n1 : 0;
                    gy -= gy >= n1 ? n1 : 0;
                    gx2 += gx2 < 0 ? n2 : 0;
                    gx2 -= gx2 >= n2 ? n2 : 0;
                    gx2 -= gx2 >= n2 ? n2 : 0;
                    pf[u] = grid[(size_t)gz * pstride + (size_t)gy * n2 + gx2];
                }
            }
        };
        auto planes_store = [&](int j0, int nz) __attribute__((always_inline)) {
            int t = tid;
            asm volatile("" : "+v"(t));
#pragma unroll
            for (int u = 0; u < NPF; ++u) {
                const int e = t + u * NTH;
                const int zz = e / PLANE, c = e - zz * PLANE;
                if (zz < nz) ring[((j0 + zz) % NP) * PLANE + c] = pf[u];
            }
        };
        // the planes before the first phase's own
        for (int j = 0; j < M2 - 1; j += DZ) {
            const int nz = min(DZ, M2 - 1 - j);
            planes_fetch(j, nz);
            planes_store(j, nz);
        }
        range(za);
        planes_fetch(M2 - 1, min(DZ, ze - za));
        for (int zc = za, jp = 0; zc < ze; zc += DZ, jp += DZ) {  // jp: first window plane of the phase's points
            planes_store(jp + M2 - 1, min(DZ, ze - zc));
            // the phase's batches, numbered line by line
            const int first = a0, cnt = a1 - a0;
            const int nb = (cnt + G - 1) / G;
            int incl = nb;
#pragma unroll
            for (int o = 1; o < NL; o <<= 1) {
                const int y = __shfl_up(incl, o, 64);
                if (lane >= o) incl += y;
            }
            const int total = __builtin_amdgcn_readlane(incl, NL - 1);
            __syncthreads();
            range(zc + DZ);
            if (zc + DZ < ze) planes_fetch(jp + DZ + M2 - 1, min(DZ, ze - zc - DZ));
            for (int t = wave; t < total; t += NW) {
                const int ln = __popcll(__ballot(lane < NL && incl <= t));
                const int b = t - (__builtin_amdgcn_readlane(incl, ln) - __builtin_amdgcn_readlane(nb, ln));
                const int p0 = __builtin_amdgcn_readlane(first, ln) + b * G;
                const int np = min(G, __builtin_amdgcn_readlane(cnt, ln) - b * G);
                const unsigned char *rp = recb + (size_t)p0 * rbytes;
                // first window planes (ring numbering) and, one per lane, the dim-0 weights
                int j1[G];
                R wz[G], dz[GRAD ? G : 1];
#pragma unroll
                for (int p = 0; p < G; ++p) {
                    const unsigned char *q = rp + (size_t)min(p, np - 1) * rbytes;
                    const R *ps = reinterpret_cast<const R *>(q);
                    wz[p] = ps[min(lane, M2 - 1)];
                    if constexpr (GRAD) dz[p] = ps[OFF_D + min(lane, M2 - 1)];
                    const int c0 = as_const(reinterpret_cast<const int *>(q + OFF_PZ))[0];
                    j1[p] = p < np ? c0 - za : 1 << 28;
                }
                const int clast = as_const(reinterpret_cast<const int *>(rp + (size_t)(np - 1) * rbytes + OFF_PZ))[0];
                const int jend = flat ? 1 - qb : clast - za + M2;
                const int base = (ln / kLineT) * P + (ln & (kLineT - 1));
                // the lane's cells of a plane: cell + k RPG P (rows past the
                // footprint's last are read from its last row)
                const int cell = base + (used ? t1 * P + t2 : 0);
                const int last = base + min(t1 + RPG * (NR - 1), M2 - 1) * P + (used ? t2 : 0);
                R sr[G][NR], si[G][NR], dr[GRAD ? G : 1][GRAD ? NR : 1], di[GRAD ? G : 1][GRAD ? NR : 1];
#pragma unroll
                for (int p = 0; p < G; ++p)
#pragma unroll
                    for (int k = 0; k < NR; ++k) {
                        sr[p][k] = si[p][k] = R(0);
                        if constexpr (GRAD) dr[p][k] = di[p][k] = R(0);
                    }
                int j = flat ? -qb : j1[0];
                int ring_p = j % NP;             // plane j's place in the ring
                int slot = (j + qb + M2) % M2;   // its weights' slot (qb > -m)
                auto read = [&](V2 (&c)[NR]) __attribute__((always_inline)) {
                    const V2 *q = ring + ring_p * PLANE;
#pragma unroll
                    for (int k = 0; k < NR; ++k) c[k] = k + 1 < NR || M2 % RPG == 0 ? q[cell + k * RPG * P] : q[last];
                    ring_p = ring_p + 1 == NP ? 0 : ring_p + 1;
                };
                auto step = [&](const V2 (&c)[NR]) __attribute__((always_inline)) {
#pragma unroll
                    for (int p = 0; p < G; ++p) {
                        if ((unsigned)(j - j1[p]) >= (unsigned)M2) continue;
                        const R w = lane_value(wz[p], slot);
#pragma unroll
                        for (int k = 0; k < NR; ++k) {
                            sr[p][k] = fma(w, c[k][0], sr[p][k]);
                            si[p][k] = fma(w, c[k][1], si[p][k]);
                        }
                        if constexpr (GRAD) {
                            const R dw = lane_value(dz[p], slot);
#pragma unroll
                            for (int k = 0; k < NR; ++k) {
                                dr[p][k] = fma(dw, c[k][0], dr[p][k]);
                                di[p][k] = fma(dw, c[k][1], di[p][k]);
                            }
                        }
                    }
                    slot = slot + 1 == M2 ? 0 : slot + 1;
                    ++j;
                };
                // two planes per round, so that the next plane's reads go to
                // the other one's registers (a plane past the last one only
                // meets windows that have ended)
                V2 ca[NR], cb[NR];
                read(ca);
                while (j < jend) {
                    read(cb);
                    step(ca);
                    read(ca);
                    step(cb);
                }
                const int j8 = lane >> 3, vq = ((j8 & 1) << 2) | (j8 & 2) | (j8 >> 2);  // value of the lane's group
                // (all of the weights' loads before their first use: one at a time
                // they took a fifth of the kernel)
                R rw1[G][NR], rw2[G], rd1[GRAD ? G : 1][GRAD ? NR : 1], rd2[GRAD ? G : 1];
#pragma unroll
                for (int p = 0; p < G; ++p) {
                    const R *ps = reinterpret_cast<const R *>(rp + (size_t)min(p, np - 1) * rbytes);
                    rw2[p] = ps[2 * M2 + t2];
                    if constexpr (GRAD) rd2[p] = ps[OFF_D + 2 * M2 + t2];
#pragma unroll
                    for (int k = 0; k < NR; ++k) {
                        const int r = min(t1 + RPG * k, M2 - 1);
                        rw1[p][k] = ps[M2 + r];
                        if constexpr (GRAD) rd1[p][k] = ps[OFF_D + M2 + r];
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (GRAD) {
#pragma unroll
                    for (int p = 0; p < G; ++p) {
                        if (p >= np) break;
                        R v[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q) v[q] = R(0);
                        const R w2 = rw2[p], dw2 = rd2[p];
#pragma unroll
                        for (int k = 0; k < NR; ++k) {
                            const R w1 = row_on(k) ? rw1[p][k] : R(0);
                            const R d1 = (row_on(k) ? rd1[p][k] : R(0)) * w2, d2 = w1 * dw2;
                            const R w12 = w1 * w2;
                            v[0] = fma(sr[p][k], w12, v[0]);
                            v[1] = fma(si[p][k], w12, v[1]);
                            v[2] = fma(dr[p][k], w12, v[2]);
                            v[3] = fma(di[p][k], w12, v[3]);
                            v[4] = fma(sr[p][k], d1, v[4]);
                            v[5] = fma(si[p][k], d1, v[5]);
                            v[6] = fma(sr[p][k], d2, v[6]);
                            v[7] = fma(si[p][k], d2, v[7]);
                        }
                        const R x0 = halve32(v[0], v[1]), x1 = halve32(v[2], v[3]);
                        const R x2 = halve32(v[4], v[5]), x3 = halve32(v[6], v[7]);
                        const R r = halve8_sum(halve16(x0, x1), halve16(x2, x3));
                        if ((lane & 7) == 0) outs[(size_t)(poff + p0 + p) * 8 + vq] = r;
                    }
                } else {
                    R v[2 * G];
#pragma unroll
                    for (int p = 0; p < G; ++p) {
                        v[2 * p] = v[2 * p + 1] = R(0);
#pragma unroll
                        for (int k = 0; k < NR; ++k) {
                            const R w12 = (row_on(k) ? rw1[p][k] : R(0)) * rw2[p];
                            v[2 * p] = fma(sr[p][k], w12, v[2 * p]);
                            v[2 * p + 1] = fma(si[p][k], w12, v[2 * p + 1]);
                        }
                    }
                    // group j of 8 lanes ends with value bitrev3(j) = 2 p + component
                    const R x0 = halve32(v[0], v[1]), x1 = halve32(v[2], v[3]);
                    const R x2 = halve32(v[4], v[5]), x3 = halve32(v[6], v[7]);
                    const R r = halve8_sum(halve16(x0, x1), halve16(x2, x3));
                    if ((lane & 7) == 0 && (vq >> 1) < np) outs[(size_t)(poff + p0) * 2 + vq] = r;
                }
            }
            __syncthreads();  // the next phase's planes replace this one's first
        }
    }
    release_queue(queue);
}

// One launch for all line-method transforms of a plan (48 float32 transforms of
// up to 32^3, 2m = 10: 1215 us in one launch each, 469 us in one).
template <typename R, int M2, bool GRAD>
static hipError_t interp_lines_m(const Xform *dxf, int B, int ngroups, int n0, int *queue, int T, const unsigned char *rec,
                                 size_t rec_bytes, const int *cs, R *outs, hipStream_t s)
{
    using LB = LineBatch<R, M2, GRAD>;
    auto kern = k_interp_lines<R, M2, GRAD>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)LB::lds);
    if (e != hipSuccess) return e;
    if (ngroups < 1) return hipSuccess;
    // plane ranges of whole phases, enough of them for a few items per
    // workgroup (each range reads 2m - 1 planes more than it has); of fewer
    // planes where these would leave workgroups out
    const int slots = cu_count() * (LB::two ? 2 : 1);
    const int phases = (n0 + LB::DZ - 1) / LB::DZ;
    int ranges = std::max(1, std::min(phases, 4 * slots / ngroups));
    const bool fine = (long long)ngroups * ranges < slots;
    if (fine) ranges = std::max(ranges, std::min((n0 + kLineZ - 1) / kLineZ, (slots + ngroups - 1) / ngroups));
    const int grid = (int)std::min<long long>(slots, (long long)ngroups * ranges);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(LB::threads), LB::lds, s, dxf, B, ngroups, ranges, fine ? 1 : 0, queue, T,
                       rec, (int)rec_bytes, cs, outs);
    return hipGetLastError();
}

}  // namespace hpnfft
