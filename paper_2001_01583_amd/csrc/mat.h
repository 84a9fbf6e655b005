// 16x16x4 matrix products of one wavefront (gfx950 matrix instructions).
#pragma once

#include <hip/hip_runtime.h>

namespace hpnfft {

// 16x16x4 matrix product on one wavefront: lane l passes A[l & 15][l >> 4]
// and B[l >> 4][l & 15].  The result rows a lane holds differ by type:
// float32 rows 4 (l >> 4) + i, float64 rows 4 i + (l >> 4) (i = 0 .. 3), all
// in column l & 15.
template <typename R> struct Mat;
template <> struct Mat<float> {
    typedef float V4 __attribute__((ext_vector_type(4)));
    __device__ static inline V4 mul(float a, float b, V4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    // (component, tap row) of matrix row r, chosen so that lane group g
    // holds component g >> 1, tap rows 4 (g & 1) .. 4 (g & 1) + 3 of a result
    __device__ static inline void row(int r, int &c, int &y)
    {
        c = r >> 3;
        y = r & 7;
    }
};
template <> struct Mat<double> {
    typedef double V4 __attribute__((ext_vector_type(4)));
    __device__ static inline V4 mul(double a, double b, V4 c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    __device__ static inline void row(int r, int &c, int &y)
    {
        c = (r >> 1) & 1;
        y = 4 * (r & 1) + (r >> 2);
    }
};

}  // namespace hpnfft
