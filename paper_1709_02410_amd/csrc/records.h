// Per-blob records consumed by the pair kernels: scaled, regularised
// position (x/a, y/a, max(z, a)/a), FP32 low parts of x and y in the FP32
// layout, then B f for each right-hand side (B = min(z/a, 1), the blob-wall
// regularisation factor), zero-padded to a 16-byte multiple.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace rpyw {

template <typename R>
constexpr int pos_slots() {
    return sizeof(R) == 4 ? 5 : 3;
}
template <typename R, int K>
constexpr int rec_w() {
    return sizeof(R) == 4 ? (5 + 3 * K + 3) / 4 * 4 : (3 + 3 * K + 1) / 2 * 2;
}

// The record of blob i (i < N) into r[0 .. recw): RHS k is read from
// F + k N 3 ([kb][N][3]); when F2 is given (kb = 2) the second RHS is read
// from F2 instead.  With a periodic cell (lx, ly > 0, units of a) x and y
// are wrapped into [0, lx) and [0, ly) first, in FP64, so that differences
// stay below one cell length.  Blobs i >= N are padding: force-free blobs
// far from everything (x = y = 1e6 a, B = 0).  *B receives the blob's B.
template <typename R>
__device__ __forceinline__ void make_record(const double* __restrict__ pos, const double* __restrict__ F, int64_t N,
                                            int kb, int recw, double inv_a, const double* __restrict__ F2, double lx,
                                            double ly, int64_t i, R* r, double* B) {
    if (i >= N) {
        for (int e = 0; e < recw; ++e) r[e] = R(0);
        r[0] = R(1e6);
        r[1] = R(1e6);
        r[2] = R(1);
        *B = 0.0;
        return;
    }
    double x = pos[3 * i] * inv_a, y = pos[3 * i + 1] * inv_a;
    const double z = pos[3 * i + 2] * inv_a;
    if (lx > 0.0) {
        x -= lx * floor(x / lx);
        y -= ly * floor(y / ly);
    }
    const double b = z < 1.0 ? z : 1.0;
    const double zt = z < 1.0 ? 1.0 : z;
    int o;
    if constexpr (sizeof(R) == 4) {
        const float xh = (float)x, yh = (float)y;
        r[0] = xh;
        r[1] = yh;
        r[2] = (float)zt;
        r[3] = (float)(x - (double)xh);
        r[4] = (float)(y - (double)yh);
        o = 5;
    } else {
        r[0] = x;
        r[1] = y;
        r[2] = zt;
        o = 3;
    }
    for (int k = 0; k < kb; ++k) {
        const double* src = (F2 && k == 1) ? F2 + i * 3 : F + (k * N + i) * 3;
        for (int c = 0; c < 3; ++c) r[o + 3 * k + c] = (R)(b * src[c]);
    }
    for (int e = o + 3 * kb; e < recw; ++e) r[e] = R(0);
    *B = b;
}

// The FP64 record of blob i for K right-hand sides of which kb are given (the
// others are zero), in registers: make_record's loops over a count known only
// at run time put its record in scratch memory.  Blobs i >= N as there.
template <int K>
struct BlobRecord {
    double x, y, z, f[3 * K];
    __device__ __forceinline__ void load(const double* __restrict__ pos, const double* __restrict__ F, int64_t N,
                                         int kb, double inv_a, int64_t i) {
        const bool pad = i >= N;
        const int64_t j = pad ? N - 1 : i;
        const double h = pos[3 * j + 2] * inv_a;
        const double b = h < 1.0 ? h : 1.0;
        x = pad ? 1e6 : pos[3 * j] * inv_a;
        y = pad ? 1e6 : pos[3 * j + 1] * inv_a;
        z = (pad || h < 1.0) ? 1.0 : h;
#pragma unroll
        for (int q = 0; q < 3 * K; ++q)
            f[q] = (pad || q / 3 >= kb) ? 0.0 : b * F[((q / 3) * N + j) * 3 + q % 3];
    }
};

// Records for blobs [0, Npad) (make_record; Npad >= N), and B when Bout is
// given.
template <typename R>
__global__ void pack_kernel(const double* __restrict__ pos, const double* __restrict__ F, int64_t N, int kb,
                            int recw, double inv_a, R* __restrict__ rec, double* __restrict__ Bout,
                            const double* __restrict__ F2, double lx, double ly, int64_t Npad) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= Npad) return;
    double b;
    make_record<R>(pos, F, N, kb, recw, inv_a, F2, lx, ly, i, rec + i * recw, &b);
    if (Bout) Bout[i] = b;
}

// The same records for blobs [0, N) in the open domain (K right-hand sides, kb
// given), through LDS: a workgroup reads the forces of kPackBlobs blobs and
// writes their records in rows.  One thread per record reads and writes with a
// stride of a record: 6.7 us for 300 blobs and 9.5 for 3000 with 16 right-hand
// sides in FP32, now 4.5 and 5.5.
constexpr int kPackBlobs = 32;
template <typename R, int K>
__global__ __launch_bounds__(256) void pack_rows_kernel(const double* __restrict__ pos, const double* __restrict__ F,
                                                        int64_t N, int kb, double inv_a, R* __restrict__ rec,
                                                        double* __restrict__ Bout) {
    constexpr int RW = rec_w<R, K>(), PW = pos_slots<R>(), T = 256;
    __shared__ __attribute__((aligned(16))) R r[kPackBlobs * RW];
    __shared__ double b[kPackBlobs];
    const int64_t i0 = (int64_t)blockIdx.x * kPackBlobs;
    const int n = (int)(N - i0 < kPackBlobs ? N - i0 : kPackBlobs), t = threadIdx.x;
    if (t < n) {
        R h[PW];
        double bt;
        make_record<R>(pos, nullptr, N, 0, PW, inv_a, nullptr, 0.0, 0.0, i0 + t, h, &bt);
#pragma unroll
        for (int e = 0; e < PW; ++e) r[t * RW + e] = h[e];
        b[t] = bt;
        Bout[i0 + t] = bt;
    }
    __syncthreads();
    for (int q = t; q < 3 * K * kPackBlobs; q += T) {
        const int k = q / (3 * kPackBlobs), e = q % (3 * kPackBlobs), j = e / 3;
        if (j < n) r[j * RW + PW + 3 * k + e % 3] = k < kb ? (R)(b[j] * F[((int64_t)k * N + i0) * 3 + e]) : R(0);
    }
    constexpr int pad = RW - PW - 3 * K;
    if constexpr (pad > 0)
        for (int q = t; q < n * pad; q += T) r[q / pad * RW + PW + 3 * K + q % pad] = R(0);
    __syncthreads();
    for (int q = t; q < n * RW; q += T) rec[i0 * RW + q] = r[q];
}

}  // namespace rpyw
