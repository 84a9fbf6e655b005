// Box method for sparse point sets: spreading (the Spreading step of
// Algorithm 2) with every workgroup owning one output box of the oversampled
// grid.  (The interpolation of such sets gathers: k_gather.hip.)
//
// At a few hundredths of a point per grid cell (the batching and Ewald
// workloads) the line sweeps spend their time per work item, not per window
// tap: a tile with a halo of 2m - 1 cells is cleared, flushed to the grid with
// one global atomic per cell (several times the grid, since neighbouring tiles
// overlap) and each point's window is retired plane by plane.  Here points are
// binned into bins of at least m cells per edge, and an output box takes the
// points of the bins around it (with periodic images): every grid cell is
// written exactly once, by its owner, with no global atomics and no clearing
// of the grid beforehand.
#include "mat.h"
#include "sweep.h"

namespace hpnfft {

constexpr int kBoxThreads = 512;

// ---------------------------------------------------------------------------
// Spread.  A workgroup owns an output box of 16^3 cells (independent of the
// bins).  A (dim 0, dim 2) plane of it is one 16 x 16 matrix; each of its eight
// wavefronts holds two planes in float64 matrix accumulators (real and
// imaginary).  The points whose windows reach the box are found in parallel:
// the bins around it form runs of sorted points (contiguous along dim 2),
// thread <-> candidate point, the accepted ones go to a list in LDS.  Every
// wavefront queues the entries that reach its planes and adds them four per
// matrix product, one point per lane group, with weights that are zero outside
// the window:
//
//   D_y[z, x] += sum_p w0_p[z] (f_p (w1_p[y] w2_p[x]))
//
// where the product in brackets is formed in the plan's own type and the sums
// in float64, rounded once: what float32 sums with their errors carried along
// (w0 applied by fma) come to.  Those sums in LDS rounded the product too where
// a swap had to be tried again, so they varied: 165,888 ions on 256^3, float32, two
// runs' grids differed by 8.9e-9 (relative l2) and these sums from any of them by
// 7.2e-9.  Ewald forces differed by 1.3e-6 to 1.8e-5 between runs, and do by 1.2e-6 to
// 1.3e-5 from these: modes next to k = 0 nearly cancel, and a unit in the last
// place of one plane's sum in the last FFT pass moves the forces by 4e-6.
// The next batch's loads are in flight while one is added.  No LDS
// accumulators, no atomics; every cell is stored once.
//
// Bound by the vector datapath, which executes the matrix products.  Measured
// against boxes of (sum, error) or float64 cells in LDS with one LDS atomic
// per tap: 165,888 ions on 256^3, float64 2m = 16 1.00 -> 0.36 ms, float32 2m
// = 8 0.45 -> 0.15 ms; 393,216 ions on 500^3, float64 4.14 -> 1.21 ms; the
// sparse transforms of a 48-transform float32 batch 0.81 -> 0.39 ms.  Tried:
// 8^3 sub-boxes in registers on the vector unit, one point at a time with
// scalar loads of its shared values (float64 0.59 ms, bound by scalar
// instructions) or vector loads (0.89 ms); float64 cells in LDS with native
// adds for float32 (0.20 ms).
constexpr int kSpreadBox = 16, kPlanes = 2;  // planes per wavefront
constexpr int kSpreadRuns = 512;

// Bin range j0 .. j0 + nj - 1 (unwrapped: bin j mod nb, shifted by n floor(j /
// nb)) of the points whose windows reach cells lo .. lo + w - 1 of a dim.
__device__ inline void reach_bins(int lo, int w, int n, int nb, int m, int *j0, int *nj)
{
    const int cl = lo - m, ch = lo + w - 1 + m;  // cells of the points (windows c - m + 1 .. c + m), m <= n / 2
    const int a = cl < 0 ? box_of(cl + n, n, nb) - nb : box_of(cl, n, nb);
    const int b = ch >= n ? box_of(ch - n, n, nb) + nb : box_of(ch, n, nb);
    *j0 = a;
    *nj = b - a + 1;
}

template <typename R>
__global__ __launch_bounds__(kBoxThreads) void k_spread_box(const Xform *__restrict__ xfs, int B, int nboxes,
                                                            int per_xcd, int m,
                                                            const unsigned char *__restrict__ rec, int rec_bytes,
                                                            const R *__restrict__ fs, const int *__restrict__ cs)
{
    static_assert(kBoxThreads / 64 * kPlanes == kSpreadBox, "a wavefront for every two planes");
    typedef R V2 __attribute__((ext_vector_type(2)));
    __shared__ int run_p0[kSpreadRuns], run_soff[kSpreadRuns + 1], run_sh[kSpreadRuns], sh_scan[36];
    __shared__ int e_pos[kBoxThreads], e_off[kBoxThreads], e_cnt[2];
    __shared__ unsigned short queue[kBoxThreads / 64][kBoxThreads];
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    // neighbouring boxes on one XCD (workgroups go round robin over them)
    const int group = (int)group_index();
    const int k8 = group / kXcds, box_i = group % kXcds * per_xcd + k8;
    if (k8 >= per_xcd || box_i >= nboxes) return;
    int bl = 0, bh = B;
    while (bh - bl > 1) {
        const int mid = (bl + bh) >> 1;
        if (xfs[mid].boff <= box_i) bl = mid;
        else bh = mid;
    }
    const Xform &X = xfs[bl];
    const int M2 = 2 * m;
    int n[3], lo[3], w[3], j0[3], nj[3];
    {
        const int b = box_i - X.boff;
        const int nb1 = (X.n[1] + kSpreadBox - 1) / kSpreadBox, nb2 = (X.n[2] + kSpreadBox - 1) / kSpreadBox;
        lo[2] = b % nb2 * kSpreadBox;
        lo[1] = b / nb2 % nb1 * kSpreadBox;
        lo[0] = b / (nb2 * nb1) * kSpreadBox;
    }
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        n[t] = X.n[t];
        w[t] = min(kSpreadBox, n[t] - lo[t]);
        reach_bins(lo[t], w[t], n[t], X.nbox[t], m, &j0[t], &nj[t]);
    }
    // runs: bin (dims 0, 1) x image along dim 2
    const int nr = nj[0] * nj[1] * 3;
    {
        int cnt = 0;
        if (tid < nr) {
            const int u2 = tid % 3 - 1, i1 = tid / 3 % nj[1], i0 = tid / (3 * nj[1]);
            int j[2] = {j0[0] + i0, j0[1] + i1}, sh = 0;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int u = j[t] < 0 ? -1 : (j[t] >= X.nbox[t] ? 1 : 0);
                j[t] -= u * X.nbox[t];
                sh |= (u + 1) << (2 * t);
            }
            const int nb2 = X.nbox[2], f = max(j0[2], u2 * nb2), l = min(j0[2] + nj[2], (u2 + 1) * nb2) - 1;
            int p0 = 0;
            if (f <= l) {
                const int *kc = cs + X.key_off + ((long long)j[0] * X.nbox[1] + j[1]) * nb2 - u2 * nb2;
                p0 = kc[f];
                cnt = kc[l + 1] - p0;
            }
            run_p0[tid] = p0;
            run_sh[tid] = sh | (u2 + 1) << 4;
        }
        int total;
        const int base = block_excl_scan(cnt, sh_scan, &total);
        if (tid < nr) run_soff[tid] = base;
        if (tid == 0) {
            run_soff[nr] = total;
            e_cnt[0] = 0;
        }
        __syncthreads();
    }
    const int S = run_soff[nr];
    const int off_pz = (int)rec_off_pz(M2, sizeof(R));
    const unsigned char *recb = rec + (size_t)X.poff * rec_bytes;
    const R *fsb = fs + 2 * X.poff;
    const int sy = wave * kPlanes;  // this wavefront's planes
    const int p4 = lane >> 4, col = lane & 15;
    using V4 = Mat<double>::V4;
    V4 re[kPlanes], im[kPlanes];
#pragma unroll
    for (int z = 0; z < kPlanes; ++z) re[z] = im[z] = V4{0, 0, 0, 0};

    // a lane's point of a batch: value, weights of row and column `col` and of
    // the planes, which of them lie in the window (bits 0, 1, 2 ..)
    struct PointData {
        V2 f;
        R w0, w2, w1[kPlanes];
        int in;
    };
    for (int c0 = 0, cur = 0; c0 < S; c0 += kBoxThreads, cur ^= 1) {
        if (c0 > 0) __syncthreads();  // every wavefront is done with the list before
        if (tid == 0) e_cnt[cur ^ 1] = 0;
        // thread <-> candidate: its window against the box
        {
            const int k = c0 + tid;
            bool in = k < S;
            int pos = 0, off = 0;
            if (in) {
                const int r = find_run(run_soff, nr, k);
                pos = run_p0[r] + (k - run_soff[r]);
                const int2 hd = *reinterpret_cast<const int2 *>(recb + (size_t)pos * rec_bytes + off_pz);
                const int cell[3] = {hd.x, hd.y >> kBoxCellBits, hd.y & ((1 << kBoxCellBits) - 1)};
                const int sh = run_sh[r];
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    // first tap, relative to the box (-(2m - 1) .. 15)
                    const int f = cell[t] + ((sh >> (2 * t) & 3) - 1) * n[t] - m + 1 - lo[t];
                    in &= f > -M2 && f < w[t];
                    off |= (f + 32 & 63) << (6 * t);
                }
            }
            const unsigned long long mask = __ballot(in);
            int base = 0;
            if (lane == 0 && mask) base = atomicAdd(&e_cnt[cur], __popcll(mask));
            base = uni(base);
            if (in) {
                const int o = base + __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
                e_pos[o] = pos;
                e_off[o] = off;
            }
        }
        __syncthreads();
        const int cnt = uni(e_cnt[cur]);
        // the entries that reach this wavefront's planes
        unsigned short *q = queue[wave];
        int nq = 0;
        for (int e0 = 0; e0 < cnt; e0 += 64) {
            const int e = e0 + lane, f1 = (e_off[min(e, cnt - 1)] >> 6 & 63) - 32;
            const bool in = e < cnt && f1 < sy + kPlanes && f1 + M2 > sy;
            const unsigned long long mask = __ballot(in);
            if (in)
                q[nq + __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u))] = (unsigned short)e;
            nq += __popcll(mask);
        }
        // (LDS operations of a wavefront complete in order)
        __builtin_amdgcn_wave_barrier();
        auto fetch = [&](int i, PointData &d) __attribute__((always_inline)) {
            const int e = q[min(i + p4, nq - 1)], pos = e_pos[e], off = e_off[e];
            const R *ps = reinterpret_cast<const R *>(recb + (size_t)(unsigned)pos * (unsigned)rec_bytes);
            const int t0 = col + 32 - (off & 63), t1 = sy + 32 - (off >> 6 & 63), t2 = col + 32 - (off >> 12 & 63);
            d.f = reinterpret_cast<const V2 *>(fsb)[(unsigned)pos];
            d.w0 = ps[min(max(t0, 0), M2 - 1)];
            d.w2 = ps[2 * M2 + min(max(t2, 0), M2 - 1)];
            d.in = ((unsigned)t0 < (unsigned)M2 && i + p4 < nq ? 1 : 0) | ((unsigned)t2 < (unsigned)M2 ? 2 : 0);
#pragma unroll
            for (int y = 0; y < kPlanes; ++y) {
                d.w1[y] = ps[M2 + min(max(t1 + y, 0), M2 - 1)];
                d.in |= (unsigned)(t1 + y) < (unsigned)M2 ? 4 << y : 0;
            }
        };
        PointData d;
        if (nq > 0) fetch(0, d);
        for (int i = 0; i < nq; i += 4) {
            const double a = d.in & 1 ? (double)d.w0 : 0.0;
            double br[kPlanes], bi[kPlanes];
#pragma unroll
            for (int y = 0; y < kPlanes; ++y) {
                const bool in = (d.in & 2) && (d.in & (4 << y));
                const R w = d.w1[y] * d.w2;
                br[y] = in ? (double)(d.f[0] * w) : 0.0;
                bi[y] = in ? (double)(d.f[1] * w) : 0.0;
            }
            if (i + 4 < nq) fetch(i + 4, d);
#pragma unroll
            for (int y = 0; y < kPlanes; ++y) {
                re[y] = Mat<double>::mul(a, br[y], re[y]);
                im[y] = Mat<double>::mul(a, bi[y], im[y]);
            }
        }
    }
    // the planes, stored once (row 4 k + p4, column col of a result)
    if (col < w[2]) {
        const gptr<V2> g = as_global(reinterpret_cast<V2 *>(X.grid));
#pragma unroll
        for (int y = 0; y < kPlanes; ++y)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int z = 4 * k + p4;
                if (z < w[0] && sy + y < w[1])
                    g[((size_t)(lo[0] + z) * n[1] + lo[1] + sy + y) * n[2] + lo[2] + col] = V2{(R)re[y][k], (R)im[y][k]};
            }
    }
}

// ---------------------------------------------------------------------------
int spread_boxes(const Xform &X)
{
    int c = 1;
    for (int t = 0; t < 3; ++t) c *= (X.n[t] + kSpreadBox - 1) / kSpreadBox;
    return c;
}

template <typename R>
hipError_t launch_spread_box(int m, const Xform *dxf, int B, int nboxes, const unsigned char *rec, size_t rec_bytes,
                             const R *fs, const int *cell_start, hipStream_t s)
{
    if (nboxes <= 0) return hipSuccess;
    const int per_xcd = (nboxes + kXcds - 1) / kXcds;
    hipLaunchKernelGGL(k_spread_box<R>, launch_grid((long long)per_xcd * kXcds, kBoxThreads), dim3(kBoxThreads), 0, s, dxf,
                       B, nboxes, per_xcd, m, rec, (int)rec_bytes, fs, cell_start);
    return hipGetLastError();
}

template hipError_t launch_spread_box<double>(int, const Xform *, int, int, const unsigned char *, size_t,
                                              const double *, const int *, hipStream_t);
template hipError_t launch_spread_box<float>(int, const Xform *, int, int, const unsigned char *, size_t,
                                             const float *, const int *, hipStream_t);

}  // namespace hpnfft
