// FFT passes over the oversampled grid (Section 2: the FFT step of the
// gridding scheme; Algorithm 2 runs a forward FFT, Algorithm 5 an inverse one)
// with the crop to I_N and the division by the window's Fourier coefficients
// ("Scaling"; "Subdividing" on the way back) fused into the first / last pass.
//
// One pass transforms all pencils along one dimension.  A workgroup runs a
// mixed-radix (8, 4, 2, 3, 5, 7) Stockham autosort FFT of `count` pencils with
// FP64 twiddles (rounded once for the float path), one or more butterflies per
// thread and stage.  The first stage takes its inputs from global memory and
// the last one stores its outputs there (only those that the next step
// needs), so LDS holds the data only between stages: a pass of s stages writes
// and reads it s - 1 times.  Stages between run in place in one buffer (each
// thread reads its butterflies' inputs into registers before any output is
// written).  Lanes run along the pencil where its elements are contiguous
// (dim 2) and across pencils otherwise, in global memory and in LDS.  Pruning
// keeps the traffic at about 2.6 grid volumes per transform instead of 6.
//
// Bound by memory where the grid is large: 402 MB of the first adjoint pass over
// 256^3 complex128 in 81 us (5.0 TB/s, the rate of a copy).  Measured against
// loading every pencil to LDS, all stages in LDS with runtime divisions, and
// storing from LDS: the six passes over 256^3 float32 326 -> 171 us, float64
// 489 -> 326 us, 500^3 float64 5.14 -> 2.83 ms, a batch of 48 float32 grids 1.70
// -> 0.73 ms, 32^3 float32 (all launch) 47 -> 29 us.  The arithmetic of a stage
// is the same wherever its inputs lie (rounded()), and so are the results, bit
// for bit.
//
// Adjoint (sign -):  grid[n0][n1][n2] --dim2--> A[n0][n1][N2] --dim1--> B[n0][N1][N2]
//                    --dim0, x 1/c_k--> fhat[N0][N1][N2]
// Forward (sign +):  fhat --x 1/c_k, pad, dim0--> B --dim1--> A --dim2--> grid
// Frequency k of a length-n transform sits at bin k mod n; the cropped
// (centred) arrays store k at k + N/2.
#include <algorithm>

#include "internal.h"

namespace hpnfft {

constexpr int kFftThreads = 256;
constexpr int kFftCap = 2048;  // complex elements per workgroup (count * n)

template <typename R> struct C2 { R x, y; };
// loads and stores through global pointers, member by member (the compiler
// merges them into one 8- or 16-byte access)
template <typename R> __device__ inline C2<R> gload(gptr<const C2<R>> p) { return C2<R>{p->x, p->y}; }
template <typename R> __device__ inline void gstore(gptr<C2<R>> p, C2<R> v)
{
    p->x = v.x;
    p->y = v.y;
}

template <typename R> __device__ inline C2<R> cmul(C2<R> a, C2<R> b)
{
    return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename R> __device__ inline C2<R> cadd(C2<R> a, C2<R> b) { return {a.x + b.x, a.y + b.y}; }
template <typename R> __device__ inline C2<R> csub(C2<R> a, C2<R> b) { return {a.x - b.x, a.y - b.y}; }
// A product that stays one: it is not contracted with a sum that follows.
template <typename R> __device__ inline C2<R> rounded(C2<R> a)
{
    asm volatile("" : "+v"(a.x), "+v"(a.y));
    return a;
}
// multiply by i*S (S = +1 or -1)
template <int S, typename R> __device__ inline C2<R> mul_is(C2<R> a) { return {-S * a.y, S * a.x}; }

// In-register DFT of length RAD with kernel exp(S 2 pi i n k / RAD).
template <int S, typename R> __device__ inline void dft2(C2<R> *v)
{
    C2<R> a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
}
template <int S, typename R> __device__ inline void dft4(C2<R> *v)
{
    C2<R> a0 = v[0], a1 = v[1], a2 = v[2], a3 = v[3];
    C2<R> s02 = cadd(a0, a2), d02 = csub(a0, a2);
    C2<R> s13 = cadd(a1, a3), d13 = mul_is<S>(csub(a1, a3));
    v[0] = cadd(s02, s13);
    v[2] = csub(s02, s13);
    v[1] = cadd(d02, d13);
    v[3] = csub(d02, d13);
}
template <int S, typename R> __device__ inline void dft8(C2<R> *v)
{
    C2<R> e[4] = {v[0], v[2], v[4], v[6]};
    C2<R> o[4] = {v[1], v[3], v[5], v[7]};
    dft4<S>(e);
    dft4<S>(o);
    const R h = (R)0.70710678118654752440;
    // w^k = exp(S 2 pi i k / 8)
    C2<R> w1 = {h, S * h}, w3 = {-h, S * h};
    C2<R> t0 = o[0], t1 = cmul(o[1], w1), t2 = mul_is<S>(o[2]), t3 = cmul(o[3], w3);
    v[0] = cadd(e[0], t0);
    v[4] = csub(e[0], t0);
    v[1] = cadd(e[1], t1);
    v[5] = csub(e[1], t1);
    v[2] = cadd(e[2], t2);
    v[6] = csub(e[2], t2);
    v[3] = cadd(e[3], t3);
    v[7] = csub(e[3], t3);
}
template <int S, typename R> __device__ inline void dft3(C2<R> *v)
{
    const R c = (R)0.86602540378443864676;  // sqrt(3)/2
    C2<R> t1 = cadd(v[1], v[2]), t2 = csub(v[1], v[2]);
    C2<R> a = {v[0].x - (R)0.5 * t1.x, v[0].y - (R)0.5 * t1.y};
    C2<R> b = {-S * c * t2.y, S * c * t2.x};  // i S (sqrt3/2) t2
    v[0] = cadd(v[0], t1);
    v[1] = cadd(a, b);
    v[2] = csub(a, b);
}

// Odd prime radix P (5 or 7) as a direct DFT: the P - 1 nontrivial outputs
// pair up as k and P - k, which share the cosine sums of v[r] + v[P - r] and
// the sine sums of v[r] - v[P - r] (cos and sin of 2 pi j / P below, j = 1 ..
// (P - 1) / 2, to 20 digits).
template <int P> struct RootsOf;
template <> struct RootsOf<5> {
    static constexpr double c[3] = {1.0, 0.30901699437494742410, -0.80901699437494742410};
    static constexpr double s[3] = {0.0, 0.95105651629515357212, 0.58778525229247312917};
};
template <> struct RootsOf<7> {
    static constexpr double c[4] = {1.0, 0.62348980185873353053, -0.22252093395631440429,
                                    -0.90096886790241912624};
    static constexpr double s[4] = {0.0, 0.78183148246802980871, 0.97492791218182360702,
                                    0.43388373911755812048};
};
template <int P, int S, typename R> __device__ inline void dft_odd(C2<R> *v)
{
    constexpr int H = (P - 1) / 2;
    C2<R> sp[H + 1], dm[H + 1];
#pragma unroll
    for (int r = 1; r <= H; ++r) {
        sp[r] = cadd(v[r], v[P - r]);
        dm[r] = csub(v[r], v[P - r]);
    }
    C2<R> out[P];
    out[0] = v[0];
#pragma unroll
    for (int r = 1; r <= H; ++r) out[0] = cadd(out[0], sp[r]);
#pragma unroll
    for (int k = 1; k <= H; ++k) {
        // exp(S 2 pi i r k / P) = cos(2 pi (rk mod P)/P) + i S sin(...)
        C2<R> a = v[0], b = {R(0), R(0)};
#pragma unroll
        for (int r = 1; r <= H; ++r) {
            int q = (r * k) % P;
            const bool neg = q > H;     // sin(2 pi q / P) = -sin(2 pi (P - q) / P)
            const int j = neg ? P - q : q;
            const R cr = (R)RootsOf<P>::c[j];
            const R sr = neg ? (R)(-RootsOf<P>::s[j]) : (R)RootsOf<P>::s[j];
            a.x += cr * sp[r].x;
            a.y += cr * sp[r].y;
            b.x += sr * dm[r].x;
            b.y += sr * dm[r].y;
        }
        // out[k] = a + i S b,  out[P - k] = a - i S b
        const C2<R> ib = mul_is<S>(b);
        out[k] = cadd(a, ib);
        out[P - k] = csub(a, ib);
    }
#pragma unroll
    for (int r = 0; r < P; ++r) v[r] = out[r];
}

struct PassGeom {
    int dim, n, N, Lin, Lout, inner;
    long long outer_len;  // number of outer indices
    bool crop;            // adjoint: keep N of n outputs
    bool roll_out, roll_in;
};

__device__ inline PassGeom pass_geom(int pass, const Xform &X)
{
    PassGeom g;
    switch (pass) {
    case P_ADJ0: g.dim = 2; g.inner = 1; g.outer_len = (long long)X.n[0] * X.n[1]; break;
    case P_ADJ1: g.dim = 1; g.inner = X.N[2]; g.outer_len = X.n[0]; break;
    case P_ADJ2: g.dim = 0; g.inner = X.N[1] * X.N[2]; g.outer_len = 1; break;
    case P_FWD0: g.dim = 0; g.inner = X.N[1] * X.N[2]; g.outer_len = 1; break;
    case P_FWD1: g.dim = 1; g.inner = X.N[2]; g.outer_len = X.n[0]; break;
    default:     g.dim = 2; g.inner = 1; g.outer_len = (long long)X.n[0] * X.n[1]; break;
    }
    g.n = X.n[g.dim];
    g.N = X.N[g.dim];
    g.crop = pass <= P_ADJ2;
    g.Lin = g.crop ? g.n : g.N;
    g.Lout = g.crop ? g.N : g.n;
    g.roll_out = pass == P_ADJ2;
    g.roll_in = pass == P_FWD0;
    return g;
}

// Source and destination arrays of a pass.
template <typename R> struct PassArrays {
    gptr<const C2<R>> src;
    gptr<C2<R>> dst;
};
template <typename R> __device__ inline PassArrays<R> pass_arrays(int pass, const Xform &X, void *fhat_base)
{
    PassArrays<R> a;
    gptr<C2<R>> fh = as_global(reinterpret_cast<C2<R> *>(fhat_base)) + X.foff;
    switch (pass) {
    case P_ADJ0: a.src = as_global((const C2<R> *)X.grid); a.dst = as_global((C2<R> *)X.tmpA); break;
    case P_ADJ1: a.src = as_global((const C2<R> *)X.tmpA); a.dst = as_global((C2<R> *)X.tmpB); break;
    case P_ADJ2: a.src = as_global((const C2<R> *)X.tmpB); a.dst = fh; break;
    case P_FWD0: a.src = fh; a.dst = as_global((C2<R> *)X.tmpB); break;
    case P_FWD1: a.src = as_global((const C2<R> *)X.tmpB); a.dst = as_global((C2<R> *)X.tmpA); break;
    default:     a.src = as_global((const C2<R> *)X.tmpA); a.dst = as_global((C2<R> *)X.grid); break;
    }
    return a;
}

// floor(a / d) for 0 <= a < 2^20 from rd = 1 / d to within 2^-22: (a + 1/2) / d
// is at least 1 / (2 d) from an integer.
__device__ inline int div_small(int a, float rd) { return (int)(((float)a + 0.5f) * rd); }

// Lanes run along the pencil (ROWS) or across pencils; SCALE: with the factors
// of the Scaling / Subdividing step (dim 0).
enum PassKind { ROWS, COLS, SCALE };

// A workgroup's pencils: element j of pencil p of the input lies at src + j
// stride + p src_p (stride 1 in ROWS, src_p 1 otherwise), the output likewise.
template <typename R> struct Pencils {
    int n, N, cnt;
    float rcnt;  // 1 / cnt
    gptr<const C2<R>> src;
    gptr<C2<R>> dst;
    int stride, src_p, dst_p;
    gptr<const double> roll0, roll1, roll2;
    int inner0, N2;
    // factor of position j (dim 0) and pencil p
    __device__ inline double factor(int j, int p) const
    {
        const int ii = inner0 + p;
        return roll0[j] * roll1[ii / N2] * roll2[ii % N2];
    }
    // LDS elements of a pencil, at most 9/8 n (see stage(): element i lies at i + i / 8)
    __host__ __device__ static inline int pad(int n) { return n + n / 8; }
};

// One Stockham stage of radix RAD: inputs from global memory (FIRST) or LDS,
// outputs to LDS or (LAST) global memory.
enum StageAt { FIRST, MIDDLE, LAST };
template <StageAt AT, int RAD, int S, PassKind KIND, typename R>
__device__ __forceinline__ void stage(const Pencils<R> &P, C2<R> *buf, const C2<R> *tw, int Ns)
{
    constexpr bool CROP = S < 0;  // adjoint passes keep N of n outputs, forward ones have N of n inputs
    constexpr int MAXB = (kFftCap + RAD * kFftThreads - 1) / (RAD * kFftThreads);  // butterflies per thread
    const int n = P.n, nb = n / RAD;
    const int total = P.cnt * nb;
    const int h0 = P.N - P.N / 2, h1 = n - P.N / 2;  // bins [h0, h1) are cropped
    const float rnb = __builtin_amdgcn_rcpf((float)nb), rNs = __builtin_amdgcn_rcpf((float)Ns);
    // LDS position of element i of pencil p: a gap of one element in 8 spreads
    // the strides of the stages over the banks
    auto at = [&](int i, int p) __attribute__((always_inline)) {
        const int k = i + (i >> 3);
        return KIND == ROWS ? p * Pencils<R>::pad(n) + k : k * P.cnt + p;
    };
    C2<R> v[MAXB][RAD];
    int pen[MAXB], jj[MAXB];
    // (an opaque thread index: the positions of every radix would otherwise be
    // kept in registers over the loop of stages)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
#pragma unroll
    for (int q = 0; q < MAXB; ++q) {
        const int t = tid + q * kFftThreads;
        if (KIND == ROWS) {
            pen[q] = div_small(t, rnb);
            jj[q] = t - pen[q] * nb;
        } else {
            jj[q] = div_small(t, P.rcnt);
            pen[q] = t - jj[q] * P.cnt;
        }
        if (t >= total) continue;
        if constexpr (AT == FIRST) {
            const gptr<const C2<R>> sp = P.src + (KIND == ROWS ? pen[q] * P.src_p : pen[q]);
#pragma unroll
            for (int r = 0; r < RAD; ++r) {
                const int bin = jj[q] + r * nb;
                if (CROP) {
                    v[q][r] = gload<R>(sp + (KIND == ROWS ? bin : (long long)bin * P.stride));
                } else {
                    v[q][r] = C2<R>{R(0), R(0)};
                    if (bin < h0 || bin >= h1) {
                        const int j = bin < h0 ? bin + P.N / 2 : bin - h1;
                        v[q][r] = gload<R>(sp + (KIND == ROWS ? j : (long long)j * P.stride));
                        if (KIND == SCALE) {
                            const double f = P.factor(j, pen[q]);
                            v[q][r] = rounded(C2<R>{(R)(v[q][r].x * f), (R)(v[q][r].y * f)});
                        }
                    }
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < RAD; ++r) v[q][r] = buf[at(jj[q] + r * nb, pen[q])];
            if (RAD > 1) {
                const int k = jj[q] - div_small(jj[q], rNs) * Ns;
                const int tstep = AT == LAST ? 1 : n / (Ns * RAD);
#pragma unroll
                for (int r = 1; r < RAD; ++r) v[q][r] = rounded(cmul(v[q][r], tw[k * r * tstep]));
            }
        }
    }
    if (AT == MIDDLE) __syncthreads();
#pragma unroll
    for (int q = 0; q < MAXB; ++q) {
        if (tid + q * kFftThreads >= total) continue;
        if (AT == FIRST && !CROP)
#pragma unroll
            for (int r = 0; r < RAD; ++r) v[q][r] = rounded(v[q][r]);
        if (RAD == 2) dft2<S>(v[q]);
        if (RAD == 3) dft3<S>(v[q]);
        if (RAD == 4) dft4<S>(v[q]);
        if (RAD == 8) dft8<S>(v[q]);
        if (RAD == 5) dft_odd<5, S>(v[q]);
        if (RAD == 7) dft_odd<7, S>(v[q]);
#pragma unroll
        for (int r = 0; r < RAD; ++r) v[q][r] = rounded(v[q][r]);
        if constexpr (AT == LAST) {
            const gptr<C2<R>> dp = P.dst + (KIND == ROWS ? pen[q] * P.dst_p : pen[q]);
#pragma unroll
            for (int r = 0; r < RAD; ++r) {
                const int bin = jj[q] + r * nb;  // (the last stage has Ns = nb)
                int o = bin;
                if (CROP) {
                    if (bin >= h0 && bin < h1) continue;
                    o = bin < h0 ? bin + P.N / 2 : bin - h1;
                }
                C2<R> w = v[q][r];
                if (CROP && KIND == SCALE) {
                    const double f = P.factor(o, pen[q]);
                    w.x = (R)(w.x * f);
                    w.y = (R)(w.y * f);
                }
                gstore<R>(dp + (KIND == ROWS ? o : (long long)o * P.stride), w);
            }
        } else {
            const int b = AT == FIRST ? jj[q] : div_small(jj[q], rNs), k = AT == FIRST ? 0 : jj[q] - b * Ns;
#pragma unroll
            for (int r = 0; r < RAD; ++r) buf[at(b * Ns * RAD + k + r * Ns, pen[q])] = v[q][r];
        }
    }
    if (AT != LAST) __syncthreads();
}

// ODD: grids with factors 5 or 7 (their stages hold more values per thread;
// the other grids run a variant without them, with fewer registers).
template <StageAt AT, int S, PassKind KIND, bool ODD, typename R>
__device__ __forceinline__ void stage_of(int rad, const Pencils<R> &P, C2<R> *buf, const C2<R> *tw, int Ns)
{
    switch (rad) {
    case 8: stage<AT, 8, S, KIND, R>(P, buf, tw, Ns); break;
    case 4: stage<AT, 4, S, KIND, R>(P, buf, tw, Ns); break;
    case 2: stage<AT, 2, S, KIND, R>(P, buf, tw, Ns); break;
    case 3: stage<AT, 3, S, KIND, R>(P, buf, tw, Ns); break;
    case 1:
        if constexpr (AT != MIDDLE) stage<AT, 1, S, KIND, R>(P, buf, tw, Ns);
        break;
    default:
        if constexpr (ODD) {
            if (rad == 5) stage<AT, 5, S, KIND, R>(P, buf, tw, Ns);
            else stage<AT, 7, S, KIND, R>(P, buf, tw, Ns);
        }
        break;
    }
}

template <typename R, int S, PassKind KIND, bool ODD>
__global__ __launch_bounds__(kFftThreads) void k_fft(int pass, const Xform *__restrict__ xfs,
                                                     const FItem *__restrict__ items, int nitems, int per_xcd,
                                                     void *fhat_base)
{
    extern __shared__ __align__(16) unsigned char smem[];
    // neighbouring items on one XCD (workgroups go round robin over them)
    const int k8 = blockIdx.x / kXcds, it = (int)(blockIdx.x % kXcds) * per_xcd + k8;
    if (k8 >= per_xcd || it >= nitems) return;
    const FItem W = items[it];
    const Xform &X = xfs[W.xf];
    const PassGeom g = pass_geom(pass, X);
    const PassArrays<R> a = pass_arrays<R>(pass, X, fhat_base);
    const int n = g.n;
    Pencils<R> P;
    P.n = n;
    P.N = g.N;
    P.cnt = W.count;
    P.rcnt = __builtin_amdgcn_rcpf((float)W.count);
    P.src = a.src + (long long)W.outer * g.Lin * g.inner + W.inner0;  // (ROWS: inner 1, inner0 0)
    P.dst = a.dst + (long long)W.outer * g.Lout * g.inner + W.inner0;
    P.stride = g.inner;
    P.src_p = g.Lin;
    P.dst_p = g.Lout;
    P.roll0 = as_global(X.roll[0]);
    P.roll1 = as_global(X.roll[1]);
    P.roll2 = as_global(X.roll[2]);
    P.inner0 = W.inner0;
    P.N2 = X.N[2];
    C2<R> *buf = reinterpret_cast<C2<R> *>(smem);
    C2<R> *tw = buf + P.cnt * Pencils<R>::pad(n);
    // twiddles exp(S 2 pi i j / n) of this dimension (the table holds
    // exp(-2 pi i j / n)); the first stage, which uses none, ends with a barrier
    const gptr<const C2<R>> twg = as_global(reinterpret_cast<const C2<R> *>(X.tw[g.dim]));
    for (int j = threadIdx.x; j < n; j += kFftThreads) {
        C2<R> w = gload<R>(twg + j);
        if (S > 0) w.y = -w.y;
        tw[j] = w;
    }
    // radix 8 first, then 4, 2, 3, 5, 7 (a single stage is followed by a copy)
    auto radix = [](int rem) __attribute__((always_inline)) {
        return (rem % 8 == 0) ? 8 : (rem % 4 == 0) ? 4 : (rem % 2 == 0) ? 2 : (rem % 3 == 0) ? 3
             : (rem % 5 == 0) ? 5 : (rem % 7 == 0) ? 7 : 1;
    };
    int rad = radix(n), Ns = rad, rem = n / rad;
    stage_of<FIRST, S, KIND, ODD, R>(rad, P, buf, tw, 1);
    for (rad = radix(rem); rem > rad; rad = radix(rem)) {
        stage_of<MIDDLE, S, KIND, ODD, R>(rad, P, buf, tw, Ns);
        Ns *= rad;
        rem /= rad;
    }
    stage_of<LAST, S, KIND, ODD, R>(rad, P, buf, tw, Ns);
}

template <typename R, int S, bool ODD>
static auto fft_kernel(int pass)
{
    return pass == P_ADJ0 || pass == P_FWD2   ? k_fft<R, S, ROWS, ODD>
           : pass == P_ADJ1 || pass == P_FWD1 ? k_fft<R, S, COLS, ODD>
                                              : k_fft<R, S, SCALE, ODD>;
}

template <typename R>
hipError_t launch_fft(int pass, const Xform *dxf, const FItem *items, int nitems, int max_n, bool odd,
                      void *fhat_base, hipStream_t s)
{
    if (nitems <= 0) return hipSuccess;
    const size_t lds = (size_t)(kFftCap + kFftCap / 8 + max_n + 16) * 2 * sizeof(R);
    const bool adj = pass <= P_ADJ2;
    auto kern = adj ? (odd ? fft_kernel<R, -1, true>(pass) : fft_kernel<R, -1, false>(pass))
                    : (odd ? fft_kernel<R, 1, true>(pass) : fft_kernel<R, 1, false>(pass));
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    const int per_xcd = (nitems + kXcds - 1) / kXcds;
    hipLaunchKernelGGL(kern, dim3((unsigned)per_xcd * kXcds), dim3(kFftThreads), lds, s, pass, dxf, items, nitems, per_xcd,
                       fhat_base);
    return hipGetLastError();
}

template hipError_t launch_fft<double>(int, const Xform *, const FItem *, int, int, bool, void *, hipStream_t);
template hipError_t launch_fft<float>(int, const Xform *, const FItem *, int, int, bool, void *, hipStream_t);

}  // namespace hpnfft
