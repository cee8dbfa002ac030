// Symmetric products with two targets per lane (FP64, open domain): each
// unordered pair is evaluated once and applied both ways, as in sym_pairs.h,
// over groups of 128 blobs.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "pair_math.h"
#include "records.h"
#include "sym_pairs.h"

namespace rpyw {

// Work item (P, d) pairs target group P with source group (P + d) mod ng, as
// in sym_kernel.  A lane of each of the four waves holds targets l and l + 64
// of P; waves 0, 1 take the first 64 sources, waves 2, 3 the others, each
// half of the 64 steps (less with nseg segments, each a workgroup of its own
// partials).  In step s a lane reads source (l + s) mod 64 and evaluates it
// against both targets, so that a record read from LDS, and the LDS additions
// of the source's sums (one wave's own slots, one lane per slot and step:
// fixed order), serve two pairs; with K = 4 those would take as long as the
// arithmetic otherwise.  The records are formed here from ps (FP), or read
// from rec (ng * 128 of them, padded as sym_kernel's).
// Diagonal items evaluate a block against itself over all ordered pairs
// (target side only) and the two blocks once.
//
// Bound by FP64 vector instructions (79, 99 and 139 per unordered pair at 1, 2
// and 4 right-hand sides, issued two pairs at a time) at large N, by the
// loads and the barriers of few items below.  Against the kernels it replaces
// (us a call): one right-hand side, sym_kernel over groups of 64 with one
// target per lane: 34.9 -> 31.0 at 3840 blobs, 113 -> 100 at 8000, 594 -> 574 at
// 20000 (kSym2MinN1, kSym2MaxN1 for the sizes outside).  Two and four right-hand
// sides, plain kernel: 58 -> 38.5 and 74 -> 54 at 3840, 1110 -> 755 and 1400 ->
// 1093 at 20000.  Four right-hand sides need the register bound of two waves
// per SIMD (one wave without it: 69 us at 3840).
constexpr int kSym2Group = 128;

// How a target of a lane meets the source block: not at all, target side
// only, both sides.
enum { kSkip = 0, kTarget = 1, kBoth = 2 };

template <int K>
struct Sym2Lane {
    static constexpr int NQ = 3 * K;
    static constexpr int RW = rec_w<double, K>();
    static constexpr int NV = RW / 2;
    SymTarget<double, K> t[2];
    double acc[2][NQ];

    // Target b's record (NV vectors).
    __device__ void set(int b, const double* r) {
        t[b].x = r[0];
        t[b].y = r[1];
        t[b].z = r[2];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            t[b].f[q / 3][q % 3] = r[3 + q];
            acc[b][q] = 0.0;
        }
    }
    // The record of blob i: formed from ps (FP), or read from rec.
    template <bool FP>
    __device__ static void fetch(const double* __restrict__ rec, const PackSrc& ps, int64_t i, double (&r)[RW]) {
        if constexpr (FP) {
            BlobRecord<K> s;
            s.load(ps.pos, ps.F, ps.N, ps.kb, ps.inv_a, i);
            r[RW - 1] = 0.0;
            r[0] = s.x;
            r[1] = s.y;
            r[2] = s.z;
#pragma unroll
            for (int q = 0; q < NQ; ++q) r[3 + q] = s.f[q];
        } else {
            const double2* g = reinterpret_cast<const double2*>(rec + i * RW);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const double2 q = g[v];
                r[2 * v] = q.x;
                r[2 * v + 1] = q.y;
            }
        }
    }

    // Steps [s0, s1) against the source block whose records start at tile and
    // whose sums start at src.
    template <int M0, int M1>
    __device__ void pass(const double2* tile, double* src, int s0, int s1) {
        constexpr int M[2] = {M0, M1};
        const int l = threadIdx.x & 63;
#pragma unroll 1
        for (int s = s0; s < s1; ++s) {
            const int j = (l + s) & 63;
            double r[RW];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const double2 q = tile[v * kSym2Group + j];
                r[2 * v] = q.x;
                r[2 * v + 1] = q.y;
            }
            double dx[2], dy[2], dz[2];
            PairGeo<double> g[2];
            PairPre<double> p[2];
            bool near = false;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                if (M[b] == kSkip) continue;
                sym_diff(t[b], r, dx[b], dy[b], dz[b]);
                g[b] = pair_geo<double>(dx[b], dy[b], dz[b], t[b].z, r[2]);
            }
            // all reciprocal square roots before any of them is used
            if constexpr (M0 != kSkip && M1 != kSkip)
                __asm__ volatile("" : "+v"(g[0].w), "+v"(g[0].ir), "+v"(g[1].w), "+v"(g[1].ir));
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                if (M[b] == kSkip) continue;
                p[b] = pair_pre<double>(g[b], dz[b], t[b].z, r[2]);
                near = near || pair_near(p[b]);
            }
            if (__builtin_amdgcn_ballot_w64(near)) {
                __asm__ volatile("" ::: "memory");  // keep this a branch: do not speculate it
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    if (M[b] != kSkip) pair_fix(p[b]);
            }
            PairCoef<double> c[2];
#pragma unroll
            for (int b = 0; b < 2; ++b)
                if (M[b] != kSkip) c[b] = pair_fin(p[b]);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                double u[3] = {0.0, 0.0, 0.0};
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    if (M[b] == kSkip) continue;
                    double* a = acc[b] + 3 * k;
                    pair_apply<double>(c[b], dx[b], dy[b], dz[b], r[3 + 3 * k], r[4 + 3 * k], r[5 + 3 * k], a[0],
                                       a[1], a[2]);
                    if (M[b] == kBoth) {
                        PairCoef<double> ct = c[b];
                        ct.kcp = c[b].kcm;
                        ct.kcm = c[b].kcp;
                        pair_apply<double>(ct, dx[b], dy[b], dz[b], t[b].f[k][0], t[b].f[k][1], t[b].f[k][2], u[0],
                                           u[1], u[2]);
                    }
                }
                if constexpr (M0 == kBoth || M1 == kBoth) {
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        __hip_atomic_fetch_add(src + (3 * k + q) * 64 + j, u[q], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
        }
    }
};

// tpart: [ng * C * nseg][3 K][128], spart: [ng * (Hmax + 1) * nseg][3 K][128]
// (the layout of sym_kernel, which sym_gather reads).
template <int K, bool FP>
__global__ __launch_bounds__(256, K == 4 ? 2 : 1) void sym2_kernel(const double* __restrict__ rec, PackSrc ps, int ng,
                                                                   int C, int ipw, int Hmax, int nseg,
                                                                   double* __restrict__ tpart,
                                                                   double* __restrict__ spart) {
    using L = Sym2Lane<K>;
    constexpr int NQ = L::NQ, G = kSym2Group;
    __shared__ double2 tile[L::NV * G];
    __shared__ double sums[4][NQ][64];  // a wave's source sums; at the end two waves' target sums
    const int g = blockIdx.x % nseg, P = blockIdx.x / nseg / C, c = blockIdx.x / nseg % C;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int blk = w >> 1, len = 32 / nseg, s0 = (2 * g + (w & 1)) * len, s1 = s0 + len;
    L me;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        double r[L::RW];
        L::template fetch<FP>(rec, ps, (int64_t)P * G + 64 * b + l, r);
        me.set(b, r);
    }
    const int H = sym_rowlen(P, ng);
    const int d0 = c * ipw, d1 = d0 + ipw - 1 < H ? d0 + ipw - 1 : H;
    for (int d = d0; d <= d1; ++d) {
        const int Q = (P + d) % ng;
        __syncthreads();
        if (threadIdx.x < G) {
            double r[L::RW];
            L::template fetch<FP>(rec, ps, (int64_t)Q * G + threadIdx.x, r);
#pragma unroll
            for (int v = 0; v < L::NV; ++v) tile[v * G + threadIdx.x] = make_double2(r[2 * v], r[2 * v + 1]);
        }
        for (int e = threadIdx.x; e < 4 * NQ * 64; e += 256) (&sums[0][0][0])[e] = 0.0;
        __syncthreads();
        const double2* tl = tile + 64 * blk;
        double* src = &sums[w][0][0];
        if (d > 0)
            me.template pass<kBoth, kBoth>(tl, src, s0, s1);
        else if (blk == 0)
            me.template pass<kTarget, kSkip>(tl, src, s0, s1);
        else
            me.template pass<kBoth, kTarget>(tl, src, s0, s1);
        __syncthreads();
        double* out = spart + (((int64_t)Q * (Hmax + 1) + d) * nseg + g) * NQ * G;
        for (int e = threadIdx.x; e < NQ * G; e += 256) {
            const int q = e / G, j = e % G, b = j >> 6;
            out[e] = sums[2 * b][q][j & 63] + sums[2 * b + 1][q][j & 63];
        }
    }
    // target sums of the four waves: (0 + 2) + (1 + 3)
    double* red = &sums[0][0][0];
    auto put = [&](double* r) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int b = 0; b < 2; ++b) r[q * G + 64 * b + l] = me.acc[b][q];
    };
    auto add = [&](const double* r) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int b = 0; b < 2; ++b) me.acc[b][q] += r[q * G + 64 * b + l];
    };
    __syncthreads();
    if (w >= 2) put(red + (w - 2) * NQ * G);
    __syncthreads();
    if (w < 2) add(red + w * NQ * G);
    __syncthreads();
    if (w == 1) put(red);
    __syncthreads();
    if (w != 0) return;
    add(red);
    put(tpart + (int64_t)blockIdx.x * NQ * G);
}

}  // namespace rpyw
