// Products of small problems in one launch (FP64, open domain): every
// workgroup sums all sources for T targets and writes their velocities, with
// no records, no partial sums and no epilogue.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "pair_math.h"
#include "records.h"
#include "wave_sums.h"

namespace rpyw {

// A wave-uniform value moved to scalar registers.
__device__ __forceinline__ double uniform_value(double v) {
    const long long b = __builtin_bit_cast(long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(b & 0xffffffffll));
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __builtin_bit_cast(double, ((long long)hi << 32) | lo);
}

// Threads take the sources j = thread (mod 256) and apply each to the T
// targets, whose coordinates and constants are uniform (scalar registers);
// two targets share an overlap branch and interleave.  Bound by FP64 vector
// instructions once there are a few waves per SIMD, by latency and the launch
// below.  The symmetric kernel halves the pairs but pays a second launch and
// the traffic of its partial sums, the plain kernel a third launch.
// One right-hand side (us a call): 26.4 -> 6.9 at 300 blobs (plain), 10.3 -> 6.8
// at 1000, 17.3 against 14.8 at 2000, 21 against 21 at 2500 (symmetric); four:
// 32 -> 10.4 at 1000 (plain), 31 against 29 at 2000.  Two targets per
// workgroup: with one the loads weigh (16.7 at 2000), with four fewer waves
// are in flight (11.7 against 9.9 at 1500).
constexpr int kDirectThreads = 256;
constexpr int kDirectTargets = 2;
template <int K, int T = kDirectTargets>
__global__ __launch_bounds__(kDirectThreads) void direct_kernel(const double* __restrict__ pos,
                                                                const double* __restrict__ F, int64_t N, int kb,
                                                                double inv_a, double mu0, double* __restrict__ U) {
    constexpr int NV = 3 * K * T, P = fold_pad(NV);
    __shared__ double red[kDirectThreads / 64][P];
    const int64_t i0 = (int64_t)blockIdx.x * T;
    double tx[T], ty[T], tz[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int64_t i = i0 + t < N ? i0 + t : N - 1;
        const double h = pos[3 * i + 2] * inv_a;
        tx[t] = uniform_value(pos[3 * i] * inv_a);
        ty[t] = uniform_value(pos[3 * i + 1] * inv_a);
        tz[t] = uniform_value(h < 1.0 ? 1.0 : h);
    }
    double acc[P];
#pragma unroll
    for (int v = 0; v < P; ++v) acc[v] = 0.0;
    for (int64_t j = threadIdx.x; j < N; j += kDirectThreads) {
        BlobRecord<K> s;
        s.load(pos, F, N, kb, inv_a, j);
        constexpr int W = T < 2 ? 1 : 2;  // targets that share a branch
#pragma unroll
        for (int t0 = 0; t0 < T; t0 += W) {
            double dx[W], dy[W], dz[W];
            PairPre<double> p[W];
            bool near = false;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                dx[w] = tx[t0 + w] - s.x;
                dy[w] = ty[t0 + w] - s.y;
                dz[w] = tz[t0 + w] - s.z;
                p[w] = pair_pre<double>(dx[w], dy[w], dz[w], tz[t0 + w], s.z);
                near = near || pair_near(p[w]);
            }
            if (__builtin_amdgcn_ballot_w64(near)) {
                __asm__ volatile("" ::: "memory");  // keep this a branch: do not speculate it
#pragma unroll
                for (int w = 0; w < W; ++w) pair_fix(p[w]);
            }
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const PairCoef<double> c = pair_fin(p[w]);
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    double* a = acc + 3 * ((t0 + w) * K + k);
                    pair_apply<double>(c, dx[w], dy[w], dz[w], s.f[3 * k], s.f[3 * k + 1], s.f[3 * k + 2], a[0], a[1],
                                       a[2]);
                }
            }
        }
    }
    wave_fold<P, 32>(acc);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    red[wave][wave_value<P>(lane)] = acc[0];  // lanes with one value write the same sum
    __syncthreads();
    const int v = threadIdx.x;
    if (v >= NV) return;
    const int t = v / (3 * K), k = v / 3 % K, c = v % 3;
    const int64_t i = i0 + t;
    if (i >= N || k >= kb) return;
    double sum = red[0][v];
#pragma unroll
    for (int w = 1; w < kDirectThreads / 64; ++w) sum += red[w][v];
    const double h = pos[3 * i + 2] * inv_a;
    U[((int64_t)k * N + i) * 3 + c] = mu0 * (h < 1.0 ? h : 1.0) * sum;
}

}  // namespace rpyw
