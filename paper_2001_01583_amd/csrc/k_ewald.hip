// Real-space Ewald sum of Eq. (11) (Section 5) with cell lists, for the
// large ionic systems of the paper's HP-ENUF timing experiment (up to
// 12 * 64^3 ions).  The reciprocal part (Eq. (12)) runs through the NFFT.
//
// The box of side L is cut into nc^3 cubic cells of side h = L / nc >= rcut,
// so every pair closer than rcut lies in the same or a neighbouring cell.
// Ions are counting-sorted by cell (count, scan, scatter, then input order
// within each cell) into one float64 (x, y, z, q) record each.  A workgroup holds the 27 neighbour cells of a
// cell in LDS; a neighbour across the periodic boundary is shifted by L on the
// way in, so every pair is seen once per ion with its nearest image.  Each ion's force
// has a single writer; the energy is reduced per workgroup in float64 and
// summed in a fixed order.
#include <algorithm>

#include "internal.h"
#include "pairs.h"

namespace hpnfft {

constexpr int kPairThreads = 1024;
constexpr int kPairGroups = 1024;  // workgroups worth having

// Boxes of many cells with few ions each take small workgroups, four of which
// run on a compute unit: a large one's wavefronts would have no ion each, while
// its tile keeps others out.  Measured, at 1, 2, 8, 16, 32 and 64 ions per cell,
// 20^3 cells: small 60, 70, 112, 202, 483 and 1637 us, large 121, 138, 177, 264, 557
// and 1600 (one thread per ion, as before either: 96, 148, 471, 971, 2042 and
// 4888).  128 threads: 46 us at 1 ion, but 9.7 ms against 7.4 where cells hold 143
// all the same (ions in a part of the box).
constexpr int kSparseThreads = 256, kSparseCap = 1024;
static bool sparse_cells(long long M, long long ncell) { return ncell >= kPairGroups && M < 32 * ncell; }

// Parts a cell's ions are split into.
static int cell_parts(long long M, int nc)
{
    const long long ncell = (long long)nc * nc * nc;
    const long long most = std::max(1LL, M / ncell / (kPairThreads / 64));  // an ion per wavefront at least
    return (int)std::max(1LL, std::min(most, (kPairGroups + ncell - 1) / ncell));
}

// Wrap into [0, L) and return the cell coordinate along one axis.
__device__ inline double wrap_box(double v, double L)
{
    v -= L * floor(v / L);
    return v >= L ? v - L : v;  // rounding can leave exactly L
}
__device__ inline int cell_axis(double v, double inv_h, int nc)
{
    const int c = (int)(v * inv_h);
    return c < 0 ? 0 : (c >= nc ? nc - 1 : c);
}

__global__ __launch_bounds__(256) void k_cells_count(const double *__restrict__ r, long long M, double L, int nc,
                                                     int *__restrict__ counts, int *__restrict__ cell,
                                                     int *__restrict__ rank)
{
    const long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= M) return;
    const double inv_h = nc / L;
    const int cx = cell_axis(wrap_box(r[3 * j], L), inv_h, nc);
    const int cy = cell_axis(wrap_box(r[3 * j + 1], L), inv_h, nc);
    const int cz = cell_axis(wrap_box(r[3 * j + 2], L), inv_h, nc);
    const int c = (cx * nc + cy) * nc + cz;
    cell[j] = c;
    rank[j] = atomicAdd(&counts[c], 1);
}

__global__ __launch_bounds__(256) void k_cells_scatter(const double *__restrict__ r, const double *__restrict__ q,
                                                       long long M, double L, const int *__restrict__ start,
                                                       const int *__restrict__ cell, const int *__restrict__ rank,
                                                       double4 *__restrict__ sorted, int *__restrict__ orig)
{
    const long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= M) return;
    const int pos = start[cell[j]] + rank[j];
    sorted[pos] = make_double4(wrap_box(r[3 * j], L), wrap_box(r[3 * j + 1], L), wrap_box(r[3 * j + 2], L), q[j]);
    orig[pos] = (int)j;
}

// The scatter's order within a cell follows its atomic ranks, which vary from
// run to run.  This pass puts each cell's ions in the order of their input
// index (rank = ions of the cell with a smaller index), so the pair sums, and
// the results bit for bit, do not depend on that order.  Work per cell is the
// square of its ion count (about 150 at the sweep's densities).
__global__ __launch_bounds__(256) void k_cells_reorder(const double4 *__restrict__ sorted_tmp,
                                                       const int *__restrict__ orig_tmp,
                                                       const int *__restrict__ start, long long ncell,
                                                       double4 *__restrict__ sorted, int *__restrict__ orig)
{
    const long long c = group_index();
    if (c >= ncell) return;
    const int s0 = start[c], s1 = start[c + 1];
    for (int i = s0 + threadIdx.x; i < s1; i += blockDim.x) {
        const int oi = orig_tmp[i];
        int r = 0;
        for (int j = s0; j < s1; ++j) r += orig_tmp[j] < oi;
        sorted[s0 + r] = sorted_tmp[i];
        orig[s0 + r] = oi;
    }
}

// U = 1/2 sum_i sum_{j != i, r_ij < rcut} q_i q_j erfc(alpha r_ij) / r_ij and
// F_i = sum_j q_i q_j [erfc(alpha r)/r + 2 alpha/sqrt(pi) exp(-alpha^2 r^2)] d_ij / r^2.
//
// Workgroup <-> (cell, part): the ions of the 27 cells around it go to LDS
// (in tiles of CAP, shifted to their image on the way in), then each
// wavefront takes every (wavefronts x parts)-th ion of the cell.  Small boxes
// have few cells (27 at L = 3 rcut), so a cell is split into parts until about
// kPairGroups workgroups run.  An ion's partial sums over later tiles are
// added by the lanes that stored the first.
//
// Bound by the float64 vector unit (pair terms, then distance tests):
// 393,216 ions, 593 partners each within the cut-off, 143 ions per cell: 8.46
// -> 2.57 ms; 6,144 ions in 27 cells: 4.90 -> 0.10 ms.
template <int THREADS, int CAP>
__global__ __launch_bounds__(THREADS) void k_cells_pairs(const double4 *__restrict__ sorted,
                                                              const int *__restrict__ orig,
                                                              const int *__restrict__ start, int nc, int parts,
                                                              double L, double alpha, double rcut2,
                                                              double *__restrict__ part,
                                                              double *__restrict__ forces)
{
    extern __shared__ __align__(16) unsigned char smem[];
    PairTileOf<CAP> &tile = *reinterpret_cast<PairTileOf<CAP> *>(smem);
    __shared__ unsigned short queues[THREADS / 64][kPairQueue];
    __shared__ double red[THREADS / 64];
    __shared__ int off[28], t0s[27];
    __shared__ double sh[27][3];
    const long long group = group_index();
    const int c = (int)(group / parts), pt = (int)(group - (long long)c * parts);
    if (c >= nc * nc * nc) return;
    const int cz = c % nc, cy = (c / nc) % nc, cx = c / (nc * nc);
    const int s0 = start[c], s1 = start[c + 1];
    const int tid = threadIdx.x, wave = tid >> 6, nw = THREADS / 64;
    if (s0 + nw * pt >= s1) {  // no ion of the cell falls to this workgroup
        if (tid == 0) part[group] = 0.0;
        return;
    }
    if (tid < 64) {
        int n = 0;
        if (tid < 27) {
            int ax = cx + tid / 9 - 1, ay = cy + (tid / 3) % 3 - 1, az = cz + tid % 3 - 1;
            double sx = 0.0, sy = 0.0, sz = 0.0;
            if (ax < 0) { ax += nc; sx = -L; } else if (ax >= nc) { ax -= nc; sx = L; }
            if (ay < 0) { ay += nc; sy = -L; } else if (ay >= nc) { ay -= nc; sy = L; }
            if (az < 0) { az += nc; sz = -L; } else if (az >= nc) { az -= nc; sz = L; }
            const int a = (ax * nc + ay) * nc + az;
            t0s[tid] = start[a];
            n = start[a + 1] - start[a];
            sh[tid][0] = sx;
            sh[tid][1] = sy;
            sh[tid][2] = sz;
        }
        if (tid == 0) off[0] = 0;
#pragma unroll
        for (int o = 1; o < 32; o <<= 1) {
            const int y = __shfl_up(n, o, 64);
            if (tid >= o) n += y;
        }
        if (tid < 27) off[tid + 1] = n;
    }
    __syncthreads();
    const int total = off[27], own = off[13] - s0;  // candidate of own-cell ion i: own + i
    const double c2 = 2.0 * alpha / sqrt(M_PI);
    double e_acc = 0.0;
    for (int t0 = 0; t0 < total; t0 += CAP) {
        const int cnt = min(CAP, total - t0);
        if (t0 > 0) __syncthreads();
        for (int k = tid; k < cnt; k += THREADS) {
            int nb = 0;
#pragma unroll
            for (int b = 16; b > 0; b >>= 1)
                if (nb + b < 27 && off[nb + b] <= t0 + k) nb += b;
            const double4 v = sorted[t0s[nb] + (t0 + k - off[nb])];
            tile.x[k] = v.x + sh[nb][0];
            tile.y[k] = v.y + sh[nb][1];
            tile.z[k] = v.z + sh[nb][2];
            tile.q[k] = v.w;
        }
        __syncthreads();
        for (int i = s0 + wave + nw * pt; i < s1; i += nw * parts) {
            PairSum s{0.0, 0.0, 0.0, 0.0};
            sweep_pairs<false>(sorted[i], own + i - t0, cnt, tile, queues[wave], rcut2, alpha, c2, L, 0.0, s);
            if (forces) store_force(s, forces + 3 * (size_t)orig[i], t0 > 0);
            e_acc += s.e;
        }
    }
    const double e = block_sum_fixed(e_acc, red);
    if (tid == 0) part[group] = e;
}

// Workspace of the cell-list sum: [starts: nc^3 + 1 ints][scan scratch]
// [cell, rank, orig, orig in scatter order: M ints each][sorted ions, and in
// scatter order: M x 32 B each][partials: nc^3 x parts doubles], each region
// 256-byte aligned.
static size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }
static size_t scan_tmp_ints(long long n)
{
    const long long nb = (n + 4095) / 4096;
    return (size_t)(nb + nb / 2048 + 64);
}
CellsLayout cells_layout(long long M, int nc)
{
    CellsLayout C{};
    const long long ncell = (long long)nc * nc * nc;
    size_t off = 0;
    C.start = off;
    off = al256(off + (size_t)(ncell + 1) * 4);
    C.scan = off;
    off = al256(off + scan_tmp_ints(ncell + 1) * 4);
    C.cell = off;
    off = al256(off + (size_t)M * 4);
    C.rank = off;
    off = al256(off + (size_t)M * 4);
    C.orig = off;
    off = al256(off + (size_t)M * 4);
    C.orig_tmp = off;
    off = al256(off + (size_t)M * 4);
    C.sorted = off;
    off = al256(off + (size_t)M * 32);
    C.sorted_tmp = off;
    off = al256(off + (size_t)M * 32);
    C.part = off;
    off = al256(off + (size_t)ncell * cell_parts(M, nc) * 8);
    C.total = off;
    return C;
}

hipError_t launch_ewald_cells(const double *r, const double *q, long long M, double L, double alpha, double rcut,
                              int nc, unsigned char *ws, double *energy, double *forces, hipStream_t s)
{
    const CellsLayout C = cells_layout(M, nc);
    const long long ncell = (long long)nc * nc * nc;
    int *start = reinterpret_cast<int *>(ws + C.start);
    hipError_t e = launch_zero(start, (size_t)(ncell + 1) * 4, s);
    if (e != hipSuccess) return e;
    const unsigned nb = (unsigned)((M + 255) / 256);
    int *cell = reinterpret_cast<int *>(ws + C.cell), *rank = reinterpret_cast<int *>(ws + C.rank);
    int *orig = reinterpret_cast<int *>(ws + C.orig), *orig_tmp = reinterpret_cast<int *>(ws + C.orig_tmp);
    double4 *sorted = reinterpret_cast<double4 *>(ws + C.sorted);
    double4 *sorted_tmp = reinterpret_cast<double4 *>(ws + C.sorted_tmp);
    double *part = reinterpret_cast<double *>(ws + C.part);
    hipLaunchKernelGGL(k_cells_count, dim3(nb), dim3(256), 0, s, r, M, L, nc, start, cell, rank);
    e = launch_scan(start, ncell + 1, reinterpret_cast<int *>(ws + C.scan), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_cells_scatter, dim3(nb), dim3(256), 0, s, r, q, M, L, start, cell, rank, sorted_tmp,
                       orig_tmp);
    hipLaunchKernelGGL(k_cells_reorder, launch_grid(ncell, 256), dim3(256), 0, s, sorted_tmp, orig_tmp, start, ncell,
                       sorted, orig);
    const int parts = cell_parts(M, nc);
    auto pairs = [&](auto kern, int threads, size_t lds) {
        e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return;
        hipLaunchKernelGGL(kern, launch_grid(ncell * parts, threads), dim3(threads), lds, s, sorted, orig, start, nc, parts, L,
                           alpha, rcut * rcut, part, forces);
        e = hipGetLastError();
    };
    if (sparse_cells(M, ncell)) pairs(k_cells_pairs<kSparseThreads, kSparseCap>, kSparseThreads, sizeof(PairTileOf<kSparseCap>));
    else pairs(k_cells_pairs<kPairThreads, kPairCap>, kPairThreads, sizeof(PairTile));
    if (e != hipSuccess) return e;
    return launch_sum_partials(part, (int)(ncell * parts), energy, s);
}

}  // namespace hpnfft
