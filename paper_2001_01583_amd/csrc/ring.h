// Ring sweeps for windows of 2m = 8 cells, on the blocked-line layout of
// sweep.h: the spread (the Spreading step of Algorithm 2, Section 3) and the
// interpolation (the Interpolating step of Algorithm 5), both as matrix-core
// contractions.
//
// A work item is a tile of 8 x 8 z-lines (eight blocks of 8 lines, one per
// tile row) restricted to a slab of Zs planes along dim 0 (a multiple of 8),
// swept in phases of 8 planes.  A block of 8 lines has a footprint of 8 tap
// rows (dim 1) by 15 columns (dim 2), padded to 16, so with the real and
// imaginary parts as rows one plane of it is a 16 x 16 matrix:
//
//   spread         D_q[(c, y), x] += sum_p (f_p[c] w1_p[y] w0_p[q]) w2_p[x]
//   interpolation  S[(c, y), p]    = sum_q sum_x G_q[(c, y), x] (w0_p[q] w2_p[x])
//
// The spread contracts four points of the block per 16x16x4 matrix
// instruction and plane; the interpolation evaluates sixteen points, four
// columns per instruction.  The points of a block are sorted by plane, so
// the points of a batch reach nearly the same planes: 8 + (span of the
// batch's first planes) instructions per four points of the spread.  Half of
// the columns multiply a zero (the window is 8 of 15 columns wide), but the
// matrix instructions do 1024 multiply-adds in 32 cycles (float32; 64 in
// float64) and need no per-point bookkeeping, where the vector unit takes
// about 3 cycles for 64 multiply-adds and issued 75 instructions per point
// visit, 32 of them multiply-adds (half on zeros too).  Float32 and float64
// matrix instructions share the vector unit's datapath: measured, a float32
// matrix instruction and eight vector instructions take 62 cycles, 35 and 22
// by themselves.  So both kernels are bound by that unit's time, matrix plus
// vector, and by the phases' barriers; the flush of the spread is 20% of it.
//
// Measured at N = 64^3, M = 2^20 (0.5 points per grid cell), against the
// vector-unit sweeps with register windows that these replaced: float32
// spread 221 -> 135 us, interpolation 151 -> 102 us; float64 (m = 4) spread
// 315 -> 248 us, interpolation 239 -> 213 us; 2^23 points, half of them in 64
// clusters, on 256^3 (float32): spread 2818 -> 1180 us (the wavefronts of an
// item cut to fewer blocks now share them).
// Tried and slower: one branch per four slots instead of per slot (135 ->
// 167 us: 25% more matrix instructions), a switch that jumps into the slots
// (the accumulators then spill), per-lane loads of each batch one batch ahead
// instead of staged records (162 us).
#pragma once

#include <type_traits>

#include "mat.h"
#include "sweep.h"

namespace hpnfft {

constexpr int kRingP = kRingT + 7;  // footprint rows (and used columns) of a tile
constexpr int kRingThreads = 512;   // eight wavefronts
constexpr int kRingWaves = kRingThreads / 64;

// The points of one block in one group of 8 base planes (the planes of the
// points' first taps, slab-relative 8 g .. 8 g + 7): up to two runs of
// sorted points, since the group may wrap past the last plane.  The runs are
// worked off in chunks of CH points; no chunk crosses from run to run.
struct RingRun {
    int pa, na, pb, nb;  // first point and length of each run
    int ua, ub;          // planes by which the run's image lies past its points
    template <int CH> __device__ inline int chunks() const { return (na + CH - 1) / CH + (nb + CH - 1) / CH; }
    template <int CH> __device__ inline void chunk(int k, int &first, int &cnt, int &u) const
    {
        const int ka = (na + CH - 1) / CH;
        const bool in_a = k < ka;
        const int o = CH * (in_a ? k : k - ka);
        first = (in_a ? pa : pb) + o;
        cnt = min(CH, (in_a ? na : nb) - o);
        u = in_a ? ua : ub;
    }
};
// c: grid plane of the group's first base plane (its point planes are c .. c
// + len - 1, mod n0; len <= 8); cs: the block's sorted offsets, 8 per plane
__device__ inline RingRun ring_run(const int *cs, int c, int len, int n0)
{
    constexpr int BW = 8;
    RingRun r;
    r.ua = c < 0 ? -n0 : (c >= n0 ? n0 : 0);
    r.ub = r.ua + n0;
    c -= r.ua;
    const int e1 = min(c + len, n0), e2 = max(c + len - n0, 0);
    const cptr<int> k = as_const(cs);
    r.pa = k[c * BW];
    r.na = k[e1 * BW] - r.pa;
    r.pb = k[0];
    r.nb = k[e2 * BW] - r.pb;
    return r;
}

// A wavefront's next points on their way to LDS: the records of up to CH
// sorted points are consecutive in memory, so 64 lanes read them as 16-byte
// units (a few whole cache lines per instruction) into registers while the
// wavefront works on the points before them, and store them as they are.
// (Per-lane loads of each batch's weights, one batch ahead, left the
// wavefronts waiting on memory: a batch is worked off in less time than a
// load takes.)
template <typename R, int CH, bool VALUES> struct RingStage {
    static constexpr int RB = (int)rec_prefix(8, sizeof(R));  // record bytes without derivatives
    static constexpr int U = RB / 16;                         // its 16-byte units
    static constexpr int NL = (CH * U + 63) / 64;
    static constexpr int F = (int)rec_off_f(8, sizeof(R));
    typedef R V2 __attribute__((ext_vector_type(2)));
    static_assert(CH <= 64, "one value per lane");
    v4u unit[NL];
    V2 value;
    // points first .. first + cnt - 1 (1 <= cnt <= CH)
    __device__ inline void load(int first, int cnt, const unsigned char *recb, int rbytes, const R *fsb, int lane)
    {
        const unsigned char *base = recb + (size_t)first * rbytes;
        if (rbytes == RB) {
#pragma unroll
            for (int k = 0; k < NL; ++k)
                unit[k] = *reinterpret_cast<const v4u *>(base + 16 * min(lane + 64 * k, cnt * U - 1));
        } else {
            // records with derivative tables: their leading bytes only
            int l = lane;
            asm volatile("" : "+v"(l));  // (keeps the divisions of this path out of the other one's registers)
#pragma unroll
            for (int k = 0; k < NL; ++k) {
                const int e = min(l + 64 * k, cnt * U - 1), pt = e / U;
                unit[k] = *reinterpret_cast<const v4u *>(base + pt * rbytes + 16 * (e - pt * U));
            }
        }
        if constexpr (VALUES) value = reinterpret_cast<const V2 *>(fsb + 2 * (size_t)first)[min(lane, cnt - 1)];
    }
    __device__ inline void store(unsigned char *st, int lane) const
    {
#pragma unroll
        for (int k = 0; k < NL; ++k)
            if (64 * k + 63 < CH * U || lane + 64 * k < CH * U) reinterpret_cast<v4u *>(st)[lane + 64 * k] = unit[k];
        if constexpr (VALUES)
            if (lane < CH) *reinterpret_cast<V2 *>(st + lane * RB + F) = value;
    }
};

// Staged records of a periodic image u planes further, where u is no multiple
// of 8: plane and dim-0 slot order of the image (slot s: plane = s mod 8).
template <typename R>
__device__ inline void ring_image(unsigned char *st, int cnt, int u, int lane)
{
    if (lane >= cnt) return;
    unsigned char *rp = st + lane * (int)rec_prefix(8, sizeof(R));
    R *ps = reinterpret_cast<R *>(rp), w[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) w[s] = ps[s];
#pragma unroll
    for (int s = 0; s < 8; ++s) ps[(s + u) & 7] = w[s];
    *reinterpret_cast<int *>(rp + rec_off_pz(8, sizeof(R))) += u;
}

constexpr int kRingChunk = 36;  // points a wavefront of the spread stages at a time

// Wavefronts per SIMD the register budgets are set for: the float32 spread
// holds 16 planes of 4 accumulators (64 registers, 128 in all), the float64
// one twice that.
template <typename R> constexpr int ring_spread_waves() { return sizeof(R) == 4 ? 4 : 2; }

// Spread.  Each wavefront owns one block (in an item cut to fewer rows,
// several wavefronts share a block's batches) and holds two groups of 8
// planes in its accumulators: the points whose first tap lies in planes 8 g
// .. 8 g + 7 reach the planes of group g and the first seven of group g + 1.
// A batch is four points, one per lane group; the record's dim-0 weights are
// in slot order (slot s: plane = s mod 8), so weight s goes to plane s of
// group g if the point starts at or before it, else to plane s of group g + 1.
// After a group the wavefronts dump its planes into LDS and all threads add
// up the overlapping rows of the eight blocks (float32 in float64, one
// rounding) and add each cell once to the grid; the second group's planes
// carry over.
template <typename R>
__global__ __launch_bounds__(kRingThreads, ring_spread_waves<R>()) void k_spread_ring(
    const Xform *__restrict__ xfs, const SItem *__restrict__ items, int nitems, int *__restrict__ queue, int Zs,
    const unsigned char *__restrict__ rec, int rbytes, const R *__restrict__ fs, const int *__restrict__ cell_start)
{
    constexpr int M2 = 8, m = 4, BW = 8;
    constexpr int OFF_PZ = (int)rec_off_pz(M2, sizeof(R));
    using V4 = typename Mat<R>::V4;
    extern __shared__ uint4 smem16[];
    // [wavefront][plane][(y >> 2, x, c)] vectors of rows y & 3
    V4 *dump = reinterpret_cast<V4 *>(smem16);
    __shared__ int s_item;
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int p4 = lane >> 4, col = lane & 15;
    int ac, ay;  // component and tap row of the lane's row of A
    Mat<R>::row(col, ac, ay);
    // the lane's vector of a dumped plane
    const int dslot = (p4 & 1) * 32 + col * 2 + (p4 >> 1);

    for (int it = next_item(queue, &s_item); it < nitems; it = next_item(queue, &s_item)) {
        const SItem W = items[uni(it)];
        const Xform *X = xfs + W.xf;
        const int n0 = X->n[0], n1 = X->n[1], n2 = X->n[2];
        const int ntx = X->ntx;
        const int X0 = (W.tile % ntx) * kRingT, Y0 = (W.tile / ntx) * kRingT;
        const int z0 = W.slab * Zs, zs = min(Zs, n0 - z0);
        const bool flat = X->flat > 0;
        const long long poff = X->poff;
        const int nrow = W.le - W.lb, wpr = kRingWaves / nrow;  // wavefronts per block
        const int row = wave / wpr, sub = wave - row * wpr;
        const int li = W.lb + row;
        const bool mine = row < nrow && Y0 + li < n1;
        const int *cs = cell_start + X->key_off + ((long long)W.tile * (kRingT * kRingT / BW) + li) * n0 * BW;
        const unsigned char *recb = rec + (size_t)poff * rbytes;
        const R *fsb = fs + 2 * poff;

        using Stage = RingStage<R, kRingChunk, true>;
        static_assert(kRingChunk * Stage::RB <= (int)(kRingZp * 64 * sizeof(V4)), "staged in the wavefront's dump area");
        unsigned char *st = reinterpret_cast<unsigned char *>(dump + wave * kRingZp * 64);

        V4 lo[8], hi[7];
#pragma unroll
        for (int s = 0; s < 8; ++s) lo[s] = V4{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < 7; ++s) hi[s] = V4{0, 0, 0, 0};

        // the points of group g (group -1 starts at plane -7: plane -8
        // reaches nothing).  A leading dim without a coordinate holds every
        // point at plane 0 with the unit impulse there: only plane 0 receives
        // anything, from the window images that start before the slab.
        auto group_run = [&](int g) __attribute__((always_inline)) {
            const int first = g < 0 ? -(M2 - 1) : kRingZp * g;
            RingRun r = ring_run(cs, first + (m - 1) + z0, min(kRingZp * (g + 1), zs) - first, n0);
            if (flat && g >= 0) r.na = r.nb = 0;
            return r;
        };
        const int ng = (zs + kRingZp - 1) / kRingZp;
        RingRun rn{};
        Stage sg;
        // loads chunk k of run r, or the first chunk of the next group's run
        auto load_next = [&](const RingRun &r, int k) __attribute__((always_inline)) {
            const bool same = k < r.chunks<kRingChunk>();
            if (!same && sub >= rn.chunks<kRingChunk>()) return;
            int first, cnt, u;
            if (same) r.chunk<kRingChunk>(k, first, cnt, u);
            else rn.chunk<kRingChunk>(sub, first, cnt, u);
            sg.load(first, cnt, recb, rbytes, fsb, lane);
        };
        if (mine) {
            rn = group_run(-1);
            load_next(rn, sub);
        }
        for (int g = -1; g < ng; ++g) {
            if (mine) {
                const RingRun r = rn;
                rn.na = rn.nb = 0;
                if (g + 1 < ng) rn = group_run(g + 1);
                const int nch = r.chunks<kRingChunk>();
                if (sub >= nch) load_next(r, nch);
                for (int ch = sub; ch < nch; ch += wpr) {
                    int first, cnt, u;
                    r.chunk<kRingChunk>(ch, first, cnt, u);
                    sg.store(st, lane);
                    if (u & 7) ring_image<R>(st, cnt, u, lane);
                    load_next(r, ch + wpr);
                    for (int c = 0; c < cnt; c += 4) {
                        const int lastp = min(cnt - 1 - c, 3);
                        const unsigned char *rp = st + (c + min(p4, lastp)) * Stage::RB;
                        const R *ps = reinterpret_cast<const R *>(rp);
                        const V4 w0a = reinterpret_cast<const V4 *>(rp)[0], w0b = reinterpret_cast<const V4 *>(rp)[1];
                        const int2 h = *reinterpret_cast<const int2 *>(rp + OFF_PZ);
                        const R f1 = ps[3 * M2 + ac] * ps[M2 + ay], w2 = ps[2 * M2 + (col & 7)];
                        // first tap plane in its group (slabs begin at multiples of 8)
                        const int db = (h.x - (m - 1)) & 7;
                        int dmin = uni(db), dmax = __builtin_amdgcn_readlane(db, 16 * lastp);
                        if (flat) {  // slot 0 of the next group only
                            dmin = 8;
                            dmax = min(dmax, 1);
                        }
                        const R a = p4 <= lastp ? f1 : R(0);
                        // column x < 8 is reached by lines j <= x, column x >= 8
                        // by lines j > x - 8 (dim 2 is stored in lane order)
                        const R b = ((col & 7) < head_line(h.y)) == (col >= 8) ? w2 : R(0);
#pragma unroll
                        for (int s = 0; s < 8; ++s) {
                            const R aw = a * (s < 4 ? w0a[s & 3] : w0b[s & 3]);
                            const bool up = s < db;  // the slot's plane lies in the next group
                            if (s >= dmin) lo[s] = Mat<R>::mul(up ? R(0) : aw, b, lo[s]);
                            if (s < 7 && s < dmax) hi[s] = Mat<R>::mul(up ? aw : R(0), b, hi[s]);
                        }
                    }
                }
            }
            if (g >= 0) {
#pragma unroll
                for (int s = 0; s < 8; ++s) dump[(wave * 8 + s) * 64 + dslot] = lo[s];
                __syncthreads();
                const size_t pstride = (size_t)n1 * n2;
                const gptr<R> grid = as_global(reinterpret_cast<R *>(X->grid));
                const int zb = z0 + kRingZp * g, zn = zs - kRingZp * g;  // (the grid's last group may hold fewer planes)
                auto cell = [&](int z, int y, int x, int c) __attribute__((always_inline)) {
                    int gy = Y0 + y - (m - 1), gx = X0 + x - (m - 1);
                    gy += gy < 0 ? n1 : 0;
                    gy -= gy >= n1 ? n1 : 0;
                    gy -= gy >= n1 ? n1 : 0;
                    gx += gx < 0 ? n2 : 0;
                    gx -= gx >= n2 ? n2 : 0;
                    gx -= gx >= n2 ? n2 : 0;
                    return ((size_t)(zb + z) * pstride + (size_t)gy * n2 + gx) * 2 + c;
                };
                auto add = [&](int z, int y, int x, int c, double v) __attribute__((always_inline)) {
                    const R q = (R)v;
                    if (q != R(0))
                        __hip_atomic_fetch_add(&grid[cell(z, y, x, c)], q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                };
                if (nrow == kRingT) {
                    // whole tile: thread <-> (plane, column, component), the
                    // lower half of the workgroup for rows 0 .. 7, the upper
                    // half for rows 8 .. 14; consecutive lanes add to
                    // consecutive reals of the grid
                    int t = tid & 255;
                    asm volatile("" : "+v"(t));  // (addresses are cheaper computed per phase than kept in registers)
                    const int c = t & 1, x = (t >> 1) & 15, z = t >> 5;
                    const V4 *dp = dump + z * 64 + x * 2 + c;
                    auto half = [&](auto H) __attribute__((always_inline)) {
                        constexpr int r0 = decltype(H)::value ? 8 : 0;
                        double out[8];
#pragma unroll
                        for (int k = 0; k < 8; ++k) out[k] = 0.0;
#pragma unroll
                        for (int l = 0; l < kRingT; ++l)
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                if (l + 4 * h + 3 < r0 || l + 4 * h >= r0 + 8) continue;
                                const V4 v = dp[l * 512 + h * 32];
#pragma unroll
                                for (int k = 0; k < 4; ++k) {
                                    const int y = l + 4 * h + k - r0;
                                    if (y >= 0 && y < 8) out[y] += (double)v[k];
                                }
                            }
                        if (x < kRingP && z < zn) {
#pragma unroll
                            for (int k = 0; k < 8; ++k)
                                if (r0 + k < kRingP) add(z, r0 + k, x, c, out[k]);
                        }
                    };
                    if (wave < kRingWaves / 2) half(std::integral_constant<bool, false>{});
                    else half(std::integral_constant<bool, true>{});
                } else {
                    const R *dr = reinterpret_cast<const R *>(dump);
                    int t = tid;
                    asm volatile("" : "+v"(t));
                    for (int i = t; i < kRingZp * kRingP * 32; i += kRingThreads) {
                        const int c = i & 1, x = (i >> 1) & 15, zy = i >> 5;
                        const int z = zy / kRingP, y = zy - z * kRingP;
                        if (x >= kRingP || z >= zn) continue;
                        double v = 0.0;
                        for (int w = 0; w < nrow * wpr; ++w) {
                            const int yy = y - (W.lb + w / wpr);
                            if (yy >= 0 && yy < M2)
                                v += (double)dr[(((w * 8 + z) * 64 + (yy >> 2) * 32 + x * 2 + c) << 2) + (yy & 3)];
                        }
                        add(z, y, x, c, v);
                    }
                }
                if (g + 1 < ng) __syncthreads();  // (the next item begins with a barrier)
            }
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                lo[s] = s < 7 ? hi[s] : V4{0, 0, 0, 0};
                if (s < 7) hi[s] = V4{0, 0, 0, 0};
            }
        }
    }
    release_queue(queue);
}

// Interpolation on the same items.  A point is evaluated by the slab that
// holds its first tap plane, in full, by one wavefront, which stores the
// result (no atomics, no clearing).  An LDS ring holds 16 planes of the
// tile's footprint: the points that start in planes 8 g .. 8 g + 7 read the
// planes up to 8 g + 14.  The next 8 planes are read from the grid into
// registers while a group is evaluated and stored once it is done.  The
// footprint rows are padded so that the 16 matrix rows a read takes (8 tap
// rows of two components, 4 columns each) lie on different LDS banks.
template <typename R> constexpr int ring_pitch() { return sizeof(R) == 4 ? 20 : 18; }
template <typename R> constexpr int ring_plane() { return kRingP * 2 * ring_pitch<R>(); }
// points a wavefront stages at a time
template <typename R> constexpr int ring_interp_chunk() { return 16; }  // (one matrix of points)
template <typename R> constexpr size_t ring_interp_lds()
{
    return (size_t)2 * kRingZp * ring_plane<R>() * sizeof(R) +
           (size_t)kRingWaves * ring_interp_chunk<R>() * rec_prefix(8, sizeof(R));
}

template <typename R>
__global__ __launch_bounds__(kRingThreads, sizeof(R) == 4 ? 6 : 4) void k_interp_ring(
    const Xform *__restrict__ xfs, const SItem *__restrict__ items, int nitems, int *__restrict__ queue, int Zs,
    const unsigned char *__restrict__ rec, int rbytes, const int *__restrict__ cell_start, R *__restrict__ outs)
{
    constexpr int M2 = 8, m = 4, BW = 8;
    constexpr int OFF_PZ = (int)rec_off_pz(M2, sizeof(R));
    constexpr int PITCH = ring_pitch<R>(), PLANE = ring_plane<R>();
    // thread <-> footprint cell (fy, fx) of every ZP-th plane from fz
    constexpr int ZP = kRingThreads / (kRingP * kRingP), NPF = kRingZp / ZP;
    static_assert(ZP * NPF == kRingZp, "whole groups of planes");
    constexpr int CH = ring_interp_chunk<R>();
    using V4 = typename Mat<R>::V4;
    extern __shared__ uint4 smem16[];
    R *ring = reinterpret_cast<R *>(smem16);  // [plane mod 16][row][component][column]
    __shared__ int s_item;
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int p16 = lane & 15, k4 = lane >> 4;
    const int fz = tid / (kRingP * kRingP), fc = tid - fz * (kRingP * kRingP);
    const int fy = fc / kRingP, fx = fc - fy * kRingP;
    int ac, ay;
    Mat<R>::row(p16, ac, ay);

    // column 15 multiplies zero weights and is never written
    for (int i = tid; i < 2 * kRingZp * PLANE; i += kRingThreads) ring[i] = R(0);

    for (int it = next_item(queue, &s_item); it < nitems; it = next_item(queue, &s_item)) {
        const SItem W = items[uni(it)];
        const Xform *X = xfs + W.xf;
        const int n0 = X->n[0], n1 = X->n[1], n2 = X->n[2];
        const int ntx = X->ntx;
        const int X0 = (W.tile % ntx) * kRingT, Y0 = (W.tile / ntx) * kRingT;
        const int z0 = W.slab * Zs, zs = min(Zs, n0 - z0);
        const bool flat = X->flat > 0;
        const long long poff = X->poff;
        const int nrow = W.le - W.lb, wpr = kRingWaves / nrow;
        const int row = wave / wpr, sub = wave - row * wpr;
        const int li = W.lb + row;
        const bool mine = row < nrow && Y0 + li < n1;
        const int *cs = cell_start + X->key_off + ((long long)W.tile * (kRingT * kRingT / BW) + li) * n0 * BW;
        const unsigned char *recb = rec + (size_t)poff * rbytes;

        // footprint cells of 8 planes, into registers and from there to LDS
        const int ry0 = W.lb, ry1 = min(W.le, n1 - Y0) + M2 - 1;  // rows the blocks reach
        const int zr = zs + M2 - 1;                                // planes their windows reach
        const size_t pstride = (size_t)n1 * n2;
        const gptr<const R> grid = as_global(reinterpret_cast<const R *>(X->grid));
        int gy = Y0 + fy - (m - 1), gx = X0 + fx - (m - 1);
        gy += gy < 0 ? n1 : 0;
        gy -= gy >= n1 ? n1 : 0;
        gy -= gy >= n1 ? n1 : 0;
        gx += gx < 0 ? n2 : 0;
        gx -= gx >= n2 ? n2 : 0;
        gx -= gx >= n2 ? n2 : 0;
        const gptr<const R> gcell = grid + 2 * ((size_t)gy * n2 + gx);
        const bool reads = fz < ZP && fy >= ry0 && fy < ry1;
        R pr[NPF], pi[NPF];
        auto planes_fetch = [&](int q0) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < NPF; ++u) {
                const int q = q0 + fz + ZP * u;
                pr[u] = pi[u] = R(0);
                if (reads && q < zr) {
                    int gz = z0 + q;  // below 2 n0
                    gz -= gz >= n0 ? n0 : 0;
                    pr[u] = gcell[2 * (size_t)gz * pstride];
                    pi[u] = gcell[2 * (size_t)gz * pstride + 1];
                }
            }
        };
        auto planes_store = [&](int q0) __attribute__((always_inline)) {
            if (fz >= ZP) return;
#pragma unroll
            for (int u = 0; u < NPF; ++u) {
                const int o = ((q0 + fz + ZP * u) & 15) * PLANE + fy * 2 * PITCH + fx;
                ring[o] = pr[u];
                ring[o + PITCH] = pi[u];
            }
        };

        using Stage = RingStage<R, CH, false>;
        unsigned char *st = reinterpret_cast<unsigned char *>(ring + 2 * kRingZp * PLANE) + wave * CH * Stage::RB;

        const int ng = (zs + kRingZp - 1) / kRingZp;
        RingRun rn{};
        Stage sg;
        auto load_next = [&](const RingRun &r, int k) __attribute__((always_inline)) {
            const bool same = k < r.chunks<CH>();
            if (!same && sub >= rn.chunks<CH>()) return;
            int first, cnt, u;
            if (same) r.chunk<CH>(k, first, cnt, u);
            else rn.chunk<CH>(sub, first, cnt, u);
            sg.load(first, cnt, recb, rbytes, nullptr, lane);
        };
        planes_fetch(0);
        if (mine) {
            rn = ring_run(cs, (m - 1) + z0, min(kRingZp, zs), n0);
            load_next(rn, sub);
        }
        planes_store(0);
        planes_fetch(kRingZp);
        for (int g = 0; g < ng; ++g) {
            planes_store(kRingZp * (g + 1));
            __syncthreads();
            if (g + 1 < ng) planes_fetch(kRingZp * (g + 2));
            if (mine) {
                const RingRun r = rn;
                rn.na = rn.nb = 0;
                if (g + 1 < ng) rn = ring_run(cs, kRingZp * (g + 1) + (m - 1) + z0, min(kRingZp, zs - kRingZp * (g + 1)), n0);
                const int nch = r.chunks<CH>();
                if (sub >= nch) load_next(r, nch);
                // planes 8 g + t: t < 8 in one half of the ring, t >= 8 in the other
                const R *ra = ring + (li + ay) * 2 * PITCH + ac * PITCH + k4;
                const R *rlo = ra + (g & 1) * kRingZp * PLANE, *rhi = ra + ((g & 1) ^ 1) * kRingZp * PLANE;
                for (int ch = sub; ch < nch; ch += wpr) {
                    int first, cnt, u;
                    r.chunk<CH>(ch, first, cnt, u);
                    sg.store(st, lane);
                    if (u & 7) ring_image<R>(st, cnt, u, lane);
                    load_next(r, ch + wpr);
                    const int lastp = cnt - 1;  // (a chunk is one batch)
                    const unsigned char *rp = st + min(p16, lastp) * Stage::RB;
                    const R *ps = reinterpret_cast<const R *>(rp);
                    const V4 w0a = reinterpret_cast<const V4 *>(rp)[0], w0b = reinterpret_cast<const V4 *>(rp)[1];
                    const V4 w1 = reinterpret_cast<const V4 *>(rp)[2 + (k4 & 1)];
                    const R w2a = ps[2 * M2 + k4], w2b = ps[2 * M2 + 4 + k4];
                    const int2 h = *reinterpret_cast<const int2 *>(rp + OFF_PZ);
                    const int db = (h.x - (m - 1)) & 7;
                    int tmin = uni(db), tmax = __builtin_amdgcn_readlane(db, lastp) + 7;
                    if (flat) tmin = tmax = 8;  // the impulse's plane only
                    // dim-2 weights of columns k4, 4 + k4, 8 + k4, 12 + k4
                    const bool ja = k4 < head_line(h.y), jb = 4 + k4 < head_line(h.y);
                    const R b0 = ja ? R(0) : w2a, b1 = jb ? R(0) : w2b;
                    const R b2 = ja ? w2a : R(0), b3 = jb ? w2b : R(0);
                    // per plane the contraction over the columns, its
                    // product with the plane's weight one plane later (a
                    // single chain of accumulators over all planes had a 30%
                    // larger rounding error)
                    V4 D[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}}, S = {0, 0, 0, 0};
                    R wp = R(0);
#pragma unroll
                    for (int t = 0; t < 15; ++t) {
                        if (t < tmin || t > tmax) continue;
                        const int s = t & 7;
                        const bool in = t < 8 ? s >= db : s < db;
                        const R *q = (t < 8 ? rlo : rhi) + s * PLANE;
                        V4 &E = D[t & 1];
                        const V4 &P = D[(t & 1) ^ 1];
                        E = Mat<R>::mul(q[0], b0, V4{0, 0, 0, 0});
                        E = Mat<R>::mul(q[4], b1, E);
                        E = Mat<R>::mul(q[8], b2, E);
                        E = Mat<R>::mul(q[12], b3, E);
#pragma unroll
                        for (int k = 0; k < 4; ++k) S[k] = fma(P[k], wp, S[k]);
                        wp = in ? (s < 4 ? w0a[s & 3] : w0b[s & 3]) : R(0);
                    }
                    const bool odd = tmax & 1;
#pragma unroll
                    for (int k = 0; k < 4; ++k) S[k] = fma(odd ? D[1][k] : D[0][k], wp, S[k]);
                    R v = S[0] * w1[0];
                    v = fma(S[1], w1[1], v);
                    v = fma(S[2], w1[2], v);
                    v = fma(S[3], w1[3], v);
                    v += __shfl_xor(v, 16, 64);  // the other four tap rows
                    if (p16 <= lastp && !(k4 & 1)) outs[2 * (poff + first + p16) + (k4 >> 1)] = v;
                }
            }
            if (g + 1 < ng) __syncthreads();
        }
    }
    release_queue(queue);
}

template <typename R>
static hipError_t spread_ring(const Xform *dxf, const SItem *items, int nitems, int *queue, Tiling t,
                              const unsigned char *rec, size_t rec_bytes, const R *fs, const int *cs, hipStream_t s)
{
    constexpr size_t lds = (size_t)kRingWaves * kRingZp * 256 * sizeof(R);
    auto kern = k_spread_ring<R>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int per_cu = ring_spread_waves<R>() * 4 / kRingWaves;
    const int grid = std::min(cu_count() * per_cu, nitems);
    if (grid < 1) return hipSuccess;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kRingThreads), lds, s, dxf, items, nitems, queue, t.Zs, rec,
                       (int)rec_bytes, fs, cs);
    return hipGetLastError();
}

template <typename R>
static hipError_t interp_ring(const Xform *dxf, const SItem *items, int nitems, int *queue, Tiling t,
                              const unsigned char *rec, size_t rec_bytes, const int *cs, R *outs, hipStream_t s)
{
    constexpr size_t lds = ring_interp_lds<R>();
    auto kern = k_interp_ring<R>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int per_cu = std::max(1, std::min(sizeof(R) == 4 ? 3 : 2, (int)((160 * 1024) / (lds + 256))));
    const int grid = std::min(cu_count() * per_cu, nitems);
    if (grid < 1) return hipSuccess;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kRingThreads), lds, s, dxf, items, nitems, queue, t.Zs, rec,
                       (int)rec_bytes, cs, outs);
    return hipGetLastError();
}

}  // namespace hpnfft
