// Sums over the lanes of a wave.
#pragma once

#include <hip/hip_runtime.h>

namespace rpyw {

// Sums of N values over the 64 lanes: in each of the first log2(P) steps (P =
// N rounded up to a power of two) a lane exchanges half of its values with
// the lane across and adds the other half, so that it ends with the whole sum
// of one value (wave_value), then the remaining steps add that one.  P - 1
// exchanges instead of the 6 N of N separate reductions.
template <int P, int M>
__device__ __forceinline__ void wave_fold(double* v) {
    static_assert(P <= 2 * M || P <= 1, "one value per lane at the end");
    if constexpr (P > 1) {
        const bool up = threadIdx.x & M;
#pragma unroll
        for (int i = 0; i < P / 2; ++i) {
            const double keep = up ? v[i + P / 2] : v[i], send = up ? v[i] : v[i + P / 2];
            v[i] = keep + __shfl_xor(send, M, 64);
        }
        wave_fold<P / 2, M / 2>(v);
    } else if constexpr (M > 0) {
        v[0] += __shfl_xor(v[0], M, 64);
        wave_fold<1, M / 2>(v);
    }
}
// The value whose sum the lane holds after wave_fold<P, 32>.
template <int P>
__device__ __forceinline__ int wave_value(int lane) {
    int v = 0;
#pragma unroll
    for (int m = 32, h = P / 2; h > 0; m >>= 1, h >>= 1) v += (lane & m) ? h : 0;
    return v;
}
constexpr int fold_pad(int n) {
    int p = 1;
    while (p < n) p <<= 1;
    return p;
}

}  // namespace rpyw
