// Dense O(N^2) products u = M(r) f of the wall-corrected RPY blob mobility
// (arXiv:1709.02410, Sec. II.A: direct summation over all blob pairs, the
// operation whose cost dominates every Brownian-dynamics step).
//
// Pipeline per pass of kb right-hand sides:
//   pack      O(N):   AoS FP64 [N][3] -> one record per blob in the kernel
//                     precision: scaled position (x, y, z~) (+ FP32 low parts
//                     of x and y), then B_j f_j for each RHS.
//   pair      O(N^2): workgroup = 256*TPL targets x one source chunk; source
//                     records are staged through LDS tiles, every lane keeps
//                     its targets' sums in registers.  FP32 sums are plain
//                     within a tile and folded into a TwoSum (hi, lo) pair
//                     after each tile.  Partial sums per source chunk go to
//                     the workspace.
//   epilogue  O(N):   fixed-order sum of the chunk partials, times
//                     mu0 * B_i, written as FP64 [N][3].
// No floating-point atomics: results are bitwise reproducible for a fixed
// launch shape.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

#include "batched_plan.h"
#include "direct_pairs.h"
#include "mat_pairs.h"
#include "pair_math.h"
#include "records.h"
#include "rpyw_internal.h"
#include "sym_multi.h"
#include "sym_pairs.h"

namespace rpyw {

namespace {

// Targets held by one lane.
template <typename R, int K, int TPL>
struct Lane {
    R x[TPL], y[TPL], z[TPL], xl[TPL], yl[TPL];
    R acc[TPL][K][3];
    R hi[TPL][K][3], lo[TPL][K][3];  // FP32 compensated running sums

    __device__ void load(const R* __restrict__ rec, int64_t first, int64_t last, int64_t tid) {
        constexpr int RW = rec_w<R, K>();
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            int64_t i = first + (int64_t)t * kBlock + tid;
            if (i >= last) i = last - 1;
            const R* r = rec + i * RW;
            x[t] = r[0];
            y[t] = r[1];
            z[t] = r[2];
            if constexpr (sizeof(R) == 4) {
                xl[t] = r[3];
                yl[t] = r[4];
            }
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    acc[t][k][c] = R(0);
                    hi[t][k][c] = R(0);
                    lo[t][k][c] = R(0);
                }
        }
    }

    // S consecutive sources from the tile, which share one overlap branch so
    // that their arithmetic interleaves; the target's sums take them in order.
    template <int S>
    __device__ __forceinline__ void sources(const R* s) {
        constexpr int RW = rec_w<R, K>(), PW = pos_slots<R>();
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            R dx[S], dy[S], dz[S];
            PairPre<R> p[S];
            bool near = false;
#pragma unroll
            for (int i = 0; i < S; ++i) {
                const R* r = s + i * RW;
                dx[i] = x[t] - r[0];
                dy[i] = y[t] - r[1];
                if constexpr (sizeof(R) == 4) {
                    dx[i] += xl[t] - r[3];
                    dy[i] += yl[t] - r[4];
                }
                dz[i] = z[t] - r[2];
                p[i] = pair_pre<R>(dx[i], dy[i], dz[i], z[t], r[2]);
                near |= pair_near(p[i]);
            }
            if (__builtin_amdgcn_ballot_w64(near)) {
                __asm__ volatile("" ::: "memory");  // keep this a branch: do not speculate it
#pragma unroll
                for (int i = 0; i < S; ++i) pair_fix(p[i]);
            }
#pragma unroll
            for (int i = 0; i < S; ++i) {
                const PairCoef<R> c = pair_fin(p[i]);
                const R* f = s + i * RW + PW;
#pragma unroll
                for (int k = 0; k < K; ++k)
                    pair_apply<R>(c, dx[i], dy[i], dz[i], f[3 * k], f[3 * k + 1], f[3 * k + 2], acc[t][k][0],
                                  acc[t][k][1], acc[t][k][2]);
            }
        }
    }

    // Sources taken together.  FP32C, 2 and 4 right-hand sides: 23.1 -> 21.0 and
    // 30.2 -> 26.4 us a call at 1000 blobs, 2.52 -> 2.50 and 3.43 -> 3.38 ms at
    // 40000; four at a time are slower from 3000 blobs on (registers).
    static constexpr int SRC = sizeof(R) == 4 && TPL == 1 ? 2 : 1;

    // Sum over sources [s0, s1) staged through the LDS tile.
    template <int TILE>
    __device__ void run(const R* __restrict__ rec, int64_t s0, int64_t s1, R* tile) {
        constexpr int RW = rec_w<R, K>();
        for (int64_t t0 = s0; t0 < s1; t0 += TILE) {
            const int n = (int)((s1 - t0) < TILE ? (s1 - t0) : TILE);
            __syncthreads();
            const R* g = rec + t0 * RW;
            for (int e = threadIdx.x; e < n * RW; e += kBlock) tile[e] = g[e];
            __syncthreads();
            int j = 0;
            for (; j + SRC <= n; j += SRC) sources<SRC>(tile + j * RW);
            if constexpr (SRC > 1)
                for (; j < n; ++j) sources<1>(tile + j * RW);
            if constexpr (sizeof(R) == 4) {
#pragma unroll
                for (int t = 0; t < TPL; ++t)
#pragma unroll
                    for (int k = 0; k < K; ++k)
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            two_sum_acc(hi[t][k][c], lo[t][k][c], acc[t][k][c]);
                            acc[t][k][c] = R(0);
                        }
            }
        }
    }

    __device__ double total(int t, int k, int c) const {
        if constexpr (sizeof(R) == 4)
            return (double)hi[t][k][c] + (double)lo[t][k][c];
        else
            return (double)acc[t][k][c];
    }
};

// Plain product: block b -> (source chunk b % splits, target block b / splits).
// With splits a multiple of 8, all workgroups of one XCD (dispatched
// round-robin by block index) read the same source chunk.
template <typename R, int K, int TPL, int TILE>
__global__ __launch_bounds__(kBlock) void pair_kernel(const R* __restrict__ rec, int64_t N, int splits,
                                                      int64_t chunk, double* __restrict__ part) {
    __shared__ __attribute__((aligned(16))) R tile[TILE * rec_w<R, K>()];
    const int b = blockIdx.x;
    const int split = b % splits;
    const int64_t first = (int64_t)(b / splits) * kBlock * TPL;
    const int64_t s0 = (int64_t)split * chunk;
    const int64_t s1 = s0 + chunk < N ? s0 + chunk : N;
    Lane<R, K, TPL> L;
    L.load(rec, first, N, threadIdx.x);
    L.template run<TILE>(rec, s0, s1, tile);
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        const int64_t i = first + (int64_t)t * kBlock + threadIdx.x;
        if (i >= N) continue;
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) part[((int64_t)(split * K + k) * 3 + c) * N + i] = L.total(t, k, c);
    }
}

// U[k][i][c] = mu0 B_i sum_s part[s][k][c][i] for k < kb, s < splits (used[i] if
// given: batched systems): kEpiParts threads per
// (blob, component q = 3 k + c) add the chunks s = u (mod kEpiParts), then the
// shares are added in order.  Bound by the reads of the partials (coalesced
// over 64 blobs).  One thread per blob for all components and chunks, as
// before, is a serial chain of 3 K splits loads on N / 256 workgroups: 179 us
// against 5.1 us at 3840 blobs, 4 right-hand sides and 60 chunks (FP64).
constexpr int kEpiParts = 8;
__global__ __launch_bounds__(64 * kEpiParts) void epilogue_kernel(const double* __restrict__ part,
                                                                  const double* __restrict__ B, int64_t N, int kdim,
                                                                  int splits, double mu0, double* __restrict__ U,
                                                                  const int* __restrict__ used = nullptr) {
    __shared__ double red[kEpiParts][64];
    const int x = threadIdx.x & 63, u = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + x;
    const int q = blockIdx.y;
    double s = 0.0;
    if (i < N) {
        const int64_t st = (int64_t)3 * kdim * N;
        const double* p = part + (int64_t)q * N + i;
        const double first = u < splits ? p[u * st] : 0.0;  // does not wait for used[i]
        if (used) splits = used[i];
        if (u < splits) s = first;
#pragma unroll 4
        for (int c = u + kEpiParts; c < splits; c += kEpiParts) s += p[c * st];
    }
    red[u][x] = s;
    __syncthreads();
    if (u != 0 || i >= N) return;
#pragma unroll
    for (int v = 1; v < kEpiParts; ++v) s += red[v][x];
    U[((int64_t)(q / 3) * N + i) * 3 + q % 3] = mu0 * B[i] * s;
}

// Batched systems: persistent workgroups take items {sys_begin, sys_end,
// target_begin, share} (batched_plan.h) from an atomic counter.  Without `part`
// an item covers all sources of its system and writes final velocities; with it
// (few items) it covers its share of them, at multiples of the tile (the FP32
// sums of a tile are the same), and writes partial sums in the layout of
// pair_kernel's, which epilogue_kernel adds up, and in used[] the number of them.
template <typename R, int K, int TPL, int TILE>
__global__ __launch_bounds__(kBlock) void batched_kernel(const R* __restrict__ rec, const int4* __restrict__ items,
                                                         int n_items, unsigned* __restrict__ counter,
                                                         const double* __restrict__ B, double mu0, int64_t Ntot,
                                                         int kb, double* __restrict__ U,
                                                         double* __restrict__ part, int* __restrict__ used) {
    __shared__ __attribute__((aligned(16))) R tile[TILE * rec_w<R, K>()];
    __shared__ int s_item;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_item = (int)atomicAdd(counter, 1u);
        __syncthreads();
        const int item = s_item;
        if (item >= n_items) break;
        const int4 it = items[item];
        Lane<R, K, TPL> L;
        L.load(rec, it.z, it.y, threadIdx.x);
        const int2 src = part_sources(it, TILE);
        L.template run<TILE>(rec, src.x, src.y, tile);
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            const int64_t i = (int64_t)it.z + (int64_t)t * kBlock + threadIdx.x;
            if (i >= it.y) continue;
            if (part) {
                const int p = it.w & 255;
                if (p == 0) used[i] = it.w >> 8;
#pragma unroll
                for (int k = 0; k < K; ++k)
#pragma unroll
                    for (int c = 0; c < 3; ++c) part[((int64_t)(p * K + k) * 3 + c) * Ntot + i] = L.total(t, k, c);
                continue;
            }
            const double sc = mu0 * B[i];
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (k < kb) U[((int64_t)k * Ntot + i) * 3 + c] = sc * L.total(t, k, c);
        }
    }
}

// ------------------------------------------------------------ symmetric product
//
// Each unordered pair is evaluated once (sym_pairs.h): the target side
// accumulates M_ij f_j, the source side M_ji f_i, which is the same block
// applied with the two off-diagonal wall coefficients exchanged.

// PER: 0 open domain; 1 pseudo-periodic; 2 pseudo-periodic with cell sides
// above 4.5 a, where only the minimum image can overlap its target (every
// other image is at least half a cell away), so the other eight skip the
// overlap branch and their arithmetic can interleave (used in FP64).
template <typename R, int K, int PER = 0>
struct ProductBody {
    static constexpr int KREC = K;
    static constexpr int NQ = 3 * K;
    static constexpr int kUnroll = PER ? 1 : 4;
    // Open domain: two sources per step sharing one overlap branch, so that
    // their arithmetic interleaves (pair2).
    static constexpr bool kDuo = !PER;
    // One source image: target side into acc and, when SYM, source side
    // (transposed block: the two off-diagonal wall coefficients exchanged)
    // into src.
    template <bool SYM>
    __device__ static void image(const SymTarget<R, K>& t, const R* r, R dx, R dy, R dz, R (&acc)[NQ],
                                 R (&src)[NQ]) {
        apply<SYM>(pair_coef<R>(dx, dy, dz, t.z, r[2]), t, r, dx, dy, dz, acc, src);
    }
    // An image that cannot overlap its target (r > 2 a): no overlap branch.
    template <bool SYM>
    __device__ static void far_image(const SymTarget<R, K>& t, const R* r, R dx, R dy, R dz, R (&acc)[NQ],
                                     R (&src)[NQ]) {
        apply<SYM>(pair_fin(pair_pre<R>(dx, dy, dz, t.z, r[2])), t, r, dx, dy, dz, acc, src);
    }
    template <bool SYM>
    __device__ static void apply(PairCoef<R> p, const SymTarget<R, K>& t, const R* r, R dx, R dy, R dz,
                                 R (&acc)[NQ], R (&src)[NQ]) {
        constexpr int PW = pos_slots<R>();
#pragma unroll
        for (int k = 0; k < K; ++k)
            pair_apply<R>(p, dx, dy, dz, r[PW + 3 * k], r[PW + 3 * k + 1], r[PW + 3 * k + 2], acc[3 * k],
                          acc[3 * k + 1], acc[3 * k + 2]);
        if constexpr (SYM) {
            const R x = p.kcp;
            p.kcp = p.kcm;
            p.kcm = x;
#pragma unroll
            for (int k = 0; k < K; ++k)
                pair_apply<R>(p, dx, dy, dz, t.f[k][0], t.f[k][1], t.f[k][2], src[3 * k], src[3 * k + 1],
                              src[3 * k + 2]);
        }
    }
    // Sources ra and rb (open domain): the source sides go to sa and sb.
    template <bool SYM>
    __device__ static void pair2(const SymTarget<R, K>& t, const R* ra, const R* rb, R (&acc)[NQ], R (&sa)[NQ],
                                 R (&sb)[NQ]) {
        R dxa, dya, dza, dxb, dyb, dzb;
        sym_diff(t, ra, dxa, dya, dza);
        sym_diff(t, rb, dxb, dyb, dzb);
        // All four reciprocal square roots are issued before any of their
        // results is used (the empty asm takes them as inputs and outputs),
        // so that their latency overlaps.
        PairGeo<R> ga = pair_geo<R>(dxa, dya, dza, t.z, ra[2]);
        PairGeo<R> gb = pair_geo<R>(dxb, dyb, dzb, t.z, rb[2]);
        __asm__ volatile("" : "+v"(ga.w), "+v"(ga.ir), "+v"(gb.w), "+v"(gb.ir));
        PairPre<R> pa = pair_pre<R>(ga, dza, t.z, ra[2]);
        PairPre<R> pb = pair_pre<R>(gb, dzb, t.z, rb[2]);
        if (__builtin_amdgcn_ballot_w64(pair_near(pa) || pair_near(pb))) {
            __asm__ volatile("" ::: "memory");  // keep this a branch: do not speculate it
            pair_fix(pa);
            pair_fix(pb);
        }
        if constexpr (SYM) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) sa[q] = sb[q] = R(0);
        }
        apply<SYM>(pair_fin(pa), t, ra, dxa, dya, dza, acc, sa);
        apply<SYM>(pair_fin(pb), t, rb, dxb, dyb, dzb, acc, sb);
    }
    // Two images of source r that share one overlap branch, with their four
    // reciprocal square roots issued before any of them is used.
    template <bool SYM>
    __device__ static void image2(const SymTarget<R, K>& t, const R* r, R dxa, R dya, R dxb, R dyb, R dz,
                                  R (&acc)[NQ], R (&src)[NQ]) {
        PairGeo<R> ga = pair_geo<R>(dxa, dya, dz, t.z, r[2]);
        PairGeo<R> gb = pair_geo<R>(dxb, dyb, dz, t.z, r[2]);
        __asm__ volatile("" : "+v"(ga.w), "+v"(ga.ir), "+v"(gb.w), "+v"(gb.ir));
        PairPre<R> pa = pair_pre<R>(ga, dz, t.z, r[2]);
        PairPre<R> pb = pair_pre<R>(gb, dz, t.z, r[2]);
        if (__builtin_amdgcn_ballot_w64(pair_near(pa) || pair_near(pb))) {
            __asm__ volatile("" ::: "memory");  // keep this a branch: do not speculate it
            pair_fix(pa);
            pair_fix(pb);
        }
        apply<SYM>(pair_fin(pa), t, r, dxa, dya, dz, acc, src);
        apply<SYM>(pair_fin(pb), t, r, dxb, dyb, dz, acc, src);
    }
    template <bool SYM>
    __device__ static void pair(const SymTarget<R, K>& t, const R* r, R (&acc)[NQ], R (&src)[NQ],
                                const Box<R>& box) {
        R dx, dy, dz;
        sym_diff(t, r, dx, dy, dz);
        if constexpr (SYM) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) src[q] = R(0);
        }
        if constexpr (!PER) {
            image<SYM>(t, r, dx, dy, dz, acc, src);
        } else {
            // Pseudo-periodic domain: the source's minimum image (records
            // are wrapped into the cell, so the shift is 0 or one cell) and
            // the 8 periodic images around it.
            const R nx = rint_(dx * box.ilx), ny = rint_(dy * box.ily);
            dx = fma_(-nx, box.lxl, fma_(-nx, box.lxh, dx));
            dy = fma_(-ny, box.lyl, fma_(-ny, box.lyh, dy));
            // image k: shift (k / 3 - 1, k % 3 - 1) cells
            auto shifted = [&](int k, R& ex, R& ey) {
                const int sx = k / 3 - 1, sy = k % 3 - 1;
                ex = sx == 0 ? dx : sx < 0 ? dx - box.lx : dx + box.lx;
                ey = sy == 0 ? dy : sy < 0 ? dy - box.ly : dy + box.ly;
            };
            if constexpr (PER == 1) {
                // images in pairs, each pair sharing one overlap branch
#pragma unroll
                for (int k = 0; k < 8; k += 2) {
                    R ea, fa, eb, fb;
                    shifted(k, ea, fa);
                    shifted(k + 1, eb, fb);
                    image2<SYM>(t, r, ea, fa, eb, fb, dz, acc, src);
                }
                R e8, f8;
                shifted(8, e8, f8);
                image<SYM>(t, r, e8, f8, dz, acc, src);
                return;
            }
#pragma unroll
            for (int sx = -1; sx <= 1; ++sx)
#pragma unroll
                for (int sy = -1; sy <= 1; ++sy) {
                    const R ex = sx == 0 ? dx : sx < 0 ? dx - box.lx : dx + box.lx;
                    const R ey = sy == 0 ? dy : sy < 0 ? dy - box.ly : dy + box.ly;
                    if (PER == 2 && (sx != 0 || sy != 0))
                        far_image<SYM>(t, r, ex, ey, dz, acc, src);
                    else
                        image<SYM>(t, r, ex, ey, dz, acc, src);
                }
        }
    }
};

// kEpiParts threads per (blob, output component q = 3k + c): each adds its
// share of the partials (sym_gather), then the shares are added in a fixed
// order.  Blocks cover 64 consecutive blobs (coalesced partial reads).
template <typename R>
__global__ __launch_bounds__(64 * kEpiParts) void sym_epilogue(const double* __restrict__ tpart,
                                                               const R* __restrict__ spart,
                                                               const double* __restrict__ B, int64_t N, int ng, int C,
                                                               int Hmax, int nseg, int K, int G, double mu0,
                                                               double* __restrict__ U,
                                                               const double* __restrict__ pos, double inv_a) {
    __shared__ double red[kEpiParts][64];
    const int x = threadIdx.x & 63, u = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + x;
    const int q = blockIdx.y;
    red[u][x] = i < N ? sym_gather<R>(tpart, spart, i, ng, C, Hmax, 3 * K, q, G, u, kEpiParts, nseg) : 0.0;
    __syncthreads();
    if (u != 0 || i >= N) return;
    double s = red[0][x];
#pragma unroll
    for (int v = 1; v < kEpiParts; ++v) s += red[v][x];
    double b;
    if (B) {
        b = B[i];
    } else {  // records formed in the pair kernel: B from the position
        const double z = pos[3 * i + 2] * inv_a;
        b = z < 1.0 ? z : 1.0;
    }
    U[((int64_t)(q / 3) * N + i) * 3 + q % 3] = mu0 * b * s;
}

// ps: the kernel forms its records from ps (groups of 64 and 128 only);
// otherwise they are read from rec.
template <typename R, int K, int PER>
hipError_t launch_sym_t(const R* rec, const SymPlan& sp, double* tpart, R* spart, const Box<R>& box, hipStream_t st,
                        const PackSrc* ps = nullptr) {
    const dim3 grid((unsigned)((int64_t)sp.ng * sp.C * sp.nseg));
    const int ipw = sp.ipw;
    const PackSrc p0 = ps ? *ps : PackSrc{};
    if (ps && sp.G != 64) return hipErrorInvalidValue;
    if (sp.G == 64 && sp.ns == 4) {
        if (ps)
            hipLaunchKernelGGL((sym_kernel<R, ProductBody<R, K, PER>, 1, 4, true>), grid, dim3(256), 0, st, rec, sp.ng,
                               sp.C, ipw, sp.Hmax, sp.nseg, tpart, spart, box, p0);
        else
            hipLaunchKernelGGL((sym_kernel<R, ProductBody<R, K, PER>, 1, 4>), grid, dim3(256), 0, st, rec, sp.ng, sp.C,
                               ipw, sp.Hmax, sp.nseg, tpart, spart, box, p0);
    } else if (sp.G == 64) {
        if (ps)
            hipLaunchKernelGGL((sym_kernel<R, ProductBody<R, K, PER>, 1, 1, true>), grid, dim3(64), 0, st, rec, sp.ng,
                               sp.C, ipw, sp.Hmax, sp.nseg, tpart, spart, box, p0);
        else
            hipLaunchKernelGGL((sym_kernel<R, ProductBody<R, K, PER>, 1>), grid, dim3(64), 0, st, rec, sp.ng, sp.C,
                               ipw, sp.Hmax, sp.nseg, tpart, spart, box, p0);
    } else {
        hipLaunchKernelGGL((sym_kernel<R, ProductBody<R, K, PER>, 4>), grid, dim3(256), 0, st, rec, sp.ng, sp.C, ipw,
                           sp.Hmax, sp.nseg, tpart, spart, box, p0, sp.tail);
    }
    return hipGetLastError();
}

// Groups of 128 (FP64, open domain).
template <int K>
hipError_t launch_sym2_t(const double* rec, const SymPlan& sp, double* tpart, double* spart, hipStream_t st,
                         const PackSrc* ps) {
    const dim3 grid((unsigned)((int64_t)sp.ng * sp.C * sp.nseg));
    if (ps)
        hipLaunchKernelGGL((sym2_kernel<K, true>), grid, dim3(256), 0, st, rec, *ps, sp.ng, sp.C, sp.ipw, sp.Hmax,
                           sp.nseg, tpart, spart);
    else if constexpr (K == 1)  // only the Krylov steps keep records, of one right-hand side
        hipLaunchKernelGGL((sym2_kernel<K, false>), grid, dim3(256), 0, st, rec, PackSrc{}, sp.ng, sp.C, sp.ipw,
                           sp.Hmax, sp.nseg, tpart, spart);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

// Kernel-side cell description in units of a (zeros for the open domain).
template <typename R>
Box<R> make_box(const Domain& dom, double a) {
    Box<R> b{};
    if (!dom.periodic()) return b;
    auto split = [](double L, R& hi, R& lo) {
        int e;
        std::frexp(L, &e);
        const double h = std::ldexp(std::nearbyint(std::ldexp(L, 12 - e)), e - 12);  // 12 significant bits
        hi = (R)h;
        lo = (R)(L - h);
    };
    const double lx = dom.lx / a, ly = dom.ly / a;
    b.lx = (R)lx;
    b.ly = (R)ly;
    split(lx, b.lxh, b.lxl);
    split(ly, b.lyh, b.lyl);
    b.ilx = (R)(1.0 / lx);
    b.ily = (R)(1.0 / ly);
    return b;
}

__global__ void zero_u32(unsigned* p) { *p = 0u; }

// ------------------------------------------------------------ dispatch

template <typename R, int K, int TPL, int TILE>
hipError_t launch_pair_t(const R* rec, int64_t N, int splits, int64_t chunk, double* part, int64_t nblocks,
                         hipStream_t st) {
    hipLaunchKernelGGL((pair_kernel<R, K, TPL, TILE>), dim3((unsigned)nblocks), dim3(kBlock), 0, st, rec, N, splits,
                       chunk, part);
    return hipGetLastError();
}

template <typename R, int K, int TPL, int TILE>
hipError_t launch_batched_t(const R* rec, const int4* items, int n_items, unsigned* counter, const double* B,
                            double mu0, int64_t Ntot, int kb, double* U, double* part, int* used, int grid,
                            hipStream_t st) {
    hipLaunchKernelGGL((batched_kernel<R, K, TPL, TILE>), dim3(grid), dim3(kBlock), 0, st, rec, items, n_items,
                       counter, B, mu0, Ntot, kb, U, part, used);
    return hipGetLastError();
}

// Source chunks of the matrix-core kernel, each shared out over sub workgroups
// of sublen sources; splits counts the shares.
struct MatSplit {
    int splits, sub, sublen;
    int64_t chunk;
};

// Records of the plain, matrix-core and batched kernels (open domain).
template <typename R>
hipError_t launch_pack_t(int K, const double* pos, const double* F, int64_t N, int kb, double a, R* rec, double* B,
                         hipStream_t st) {
    auto rows = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((N + kPackBlobs - 1) / kPackBlobs)), dim3(256), 0, st, pos, F, N, kb,
                           1.0 / a, rec, B);
    };
    if (K == 16)
        rows(pack_rows_kernel<R, 16>);
    else if (K == 8)
        rows(pack_rows_kernel<R, 8>);
    else if (K == 4)
        rows(pack_rows_kernel<R, 4>);
    else
        hipLaunchKernelGGL(pack_kernel<R>, dim3((unsigned)((N + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, pos, F, N,
                           kb, K == 2 ? rec_w<R, 2>() : rec_w<R, 1>(), 1.0 / a, rec, B, nullptr, 0.0, 0.0, N);
    return hipGetLastError();
}
hipError_t launch_pack(int prec, int K, const double* pos, const double* F, int64_t N, int kb, double a, void* rec,
                       double* B, hipStream_t st) {
    return prec == RPYW_FP32C ? launch_pack_t<float>(K, pos, F, N, kb, a, (float*)rec, B, st)
                              : launch_pack_t<double>(K, pos, F, N, kb, a, (double*)rec, B, st);
}

template <typename R, int K>
hipError_t launch_mat_t(const void* rec, int64_t N, const MatSplit& ms, double* part, int64_t nblocks,
                        hipStream_t st) {
    hipLaunchKernelGGL((mat_pair_kernel<R, K>), dim3((unsigned)nblocks), dim3(kBlock), 0, st, (const R*)rec, N,
                       ms.splits, ms.chunk, ms.sub, ms.sublen, part);
    return hipGetLastError();
}

template <typename R, int K>
hipError_t launch_mat_batched_t(const void* rec, const int4* items, int n_items, unsigned* counter,
                                const double* B, double mu0, int64_t Ntot, int kb, double* U, double* part,
                                int* used, int grid, hipStream_t st) {
    hipLaunchKernelGGL((mat_batched_kernel<R, K>), dim3(grid), dim3(kBlock), 0, st, (const R*)rec, items, n_items,
                       counter, B, mu0, Ntot, kb, U, part, used);
    return hipGetLastError();
}

// The matrix-core launches for a precision and a block of 8 or 16.
hipError_t launch_mat(int prec, int K, const void* rec, int64_t N, const MatSplit& ms, double* part,
                      int64_t nblocks, hipStream_t st) {
    if (prec == RPYW_FP32C)
        return K == 16 ? launch_mat_t<float, 16>(rec, N, ms, part, nblocks, st)
                       : launch_mat_t<float, 8>(rec, N, ms, part, nblocks, st);
    return K == 16 ? launch_mat_t<double, 16>(rec, N, ms, part, nblocks, st)
                   : launch_mat_t<double, 8>(rec, N, ms, part, nblocks, st);
}

hipError_t launch_mat_batched(int prec, int K, const void* rec, const int4* items, int n_items, unsigned* counter,
                              const double* B, double mu0, int64_t Ntot, int kb, double* U, double* part, int* used,
                              int grid, hipStream_t st) {
    if (prec == RPYW_FP32C)
        return K == 16 ? launch_mat_batched_t<float, 16>(rec, items, n_items, counter, B, mu0, Ntot, kb, U, part, used, grid, st)
                       : launch_mat_batched_t<float, 8>(rec, items, n_items, counter, B, mu0, Ntot, kb, U, part, used, grid, st);
    return K == 16 ? launch_mat_batched_t<double, 16>(rec, items, n_items, counter, B, mu0, Ntot, kb, U, part, used, grid, st)
                   : launch_mat_batched_t<double, 8>(rec, items, n_items, counter, B, mu0, Ntot, kb, U, part, used, grid, st);
}

// Expand (K, TPL, TILE) runtime values into template instantiations.
#define RPYW_DISPATCH(R, K, TPL, TILE, FN, ...)                                   \
    [&]() -> hipError_t {                                                         \
        auto tiles = [&](auto kc, auto tc) -> hipError_t {                        \
            constexpr int KK = decltype(kc)::value;                               \
            constexpr int TT = decltype(tc)::value;                               \
            if ((TILE) == 64) return FN<R, KK, TT, 64>(__VA_ARGS__);              \
            return FN<R, KK, TT, 256>(__VA_ARGS__);                               \
        };                                                                        \
        auto tpls = [&](auto kc) -> hipError_t {                                  \
            if ((TPL) == 2) return tiles(kc, std::integral_constant<int, 2>{});   \
            return tiles(kc, std::integral_constant<int, 1>{});                   \
        };                                                                        \
        auto one = [&](auto kc) -> hipError_t {                                   \
            return tiles(kc, std::integral_constant<int, 1>{});                   \
        };                                                                        \
        switch (K) {                                                              \
            case 1: return tpls(std::integral_constant<int, 1>{});                \
            case 2: return tpls(std::integral_constant<int, 2>{});                \
            case 4: return tpls(std::integral_constant<int, 4>{});                \
            case 8: return one(std::integral_constant<int, 8>{});                 \
            default:                                                              \
                if constexpr (sizeof(R) == 8) return one(std::integral_constant<int, 8>{}); \
                else return one(std::integral_constant<int, 16>{});               \
        }                                                                         \
    }()

int pow2ceil(int k) {
    int p = 1;
    while (p < k) p <<= 1;
    return p;
}

// RHS block width of the kernel instantiation that serves kb right-hand
// sides (on the vector units FP64 stops at 8: wider blocks do not fit the
// register file; the matrix-core kernel takes 16 in both precisions).
int kernel_k(int kb, int prec, int mat) {
    return std::min(pow2ceil(kb), (prec == RPYW_FP32C || mat) ? 16 : 8);
}

// The launch shape the dispatch actually instantiates: blocks of 8 or more
// right-hand sides run one target per lane, tiles are 64 or 256.
Shape normalized(Shape s, int K, int prec) {
    (void)prec;
    s.mat = (s.mat && K >= 8) ? 1 : 0;
    if (K >= 8) s.tpl = 1;
    if (K > 4) s.sym = 0;
    if (s.ipw < 1) s.ipw = 4;
    s.tpl = s.tpl == 2 ? 2 : 1;
    s.tile = s.tile == 64 ? 64 : 256;
    return s;
}

double mu0_of(double a, double eta) { return 1.0 / (6.0 * M_PI * eta * a); }

}  // namespace

// ------------------------------------------------------------ host side

SymPlan sym_plan(int64_t N, int prec, int K, int ipw, int G) {
    SymPlan s{};
    s.G = G == 64 || G == 128 ? G : 256;
    s.ng = (int)((N + s.G - 1) / s.G);
    s.Hmax = s.ng / 2;
    if (ipw < 1) ipw = 1;
    // The target partials of groups of 128 are kept to a quarter of the
    // source partials on large problems.
    if (s.G == 128 && N > kSym2MaxN1) ipw = std::max(ipw, 4);
    s.ipw = ipw;
    s.tail = sym_tail(s.G, ipw, s.ng, s.Hmax);
    s.C = sym_chunks(ipw, s.Hmax, s.tail);
    // Segments: enough work items to give every SIMD several (independent
    // of ipw, so that the workspace bound taken at ipw 1 holds).
    const int64_t items = (int64_t)s.ng * (s.Hmax + 1);
    s.ns = s.nseg = 1;
    if (s.G == 128) {
        // An item is four waves of 32 double steps.  Segments until more than
        // half of the CUs have one: 1500 blobs (84 items, one and two
        // right-hand sides) 20.7 -> 14.2 and 24 -> 16.6 us, 2000 (144) 20.9 -> 19.4
        // and 24.5 -> 23.1; 3840 (480) 30.9 -> 32.4 and 38.5 -> 42.5.
        while (s.nseg < 4 && items * s.nseg < 160) s.nseg *= 2;
    } else {
        // Groups of 64 split the passes of few items over 4 waves of one
        // workgroup first (their sums meet in LDS), and over workgroups (each
        // with partials of its own) only when there are fewer than half as
        // many waves as wanted.
        s.ns = (s.G == 64 && items < kSymItemsMin) ? 4 : 1;
        const int64_t want = s.ns > 1 ? kSymItemsMin / 2 : kSymItemsMin;
        while (s.nseg < 4 && items * s.ns * s.nseg < want) s.nseg *= 2;
        if (s.G == 64) sym_split_override(&s.ns, &s.nseg);
    }
    const size_t npad = (size_t)s.ng * s.G;
    s.rec_bytes = align_up(npad * rec_width(prec, K) * real_size(prec)) + align_up(npad * sizeof(double));
    s.tpart_bytes = align_up((size_t)s.ng * s.C * s.nseg * 3 * K * s.G * sizeof(double));
    s.spart_bytes = align_up((size_t)s.ng * (s.Hmax + 1) * s.nseg * 3 * K * s.G * real_size(prec));
    s.ok = K <= 4 && s.spart_bytes <= kSymPartialMaxBytes && s.tpart_bytes <= kSymPartialMaxBytes &&
           (s.G != 64 || N <= kSym64MaxN);
    if (s.G == 128) {
        // Two items run on a compute unit at a time and the time goes up in steps
        // of 256 of them: a third round that is less than half full (3969 to 4480
        // blobs, one right-hand side) leaves groups of 64 ahead, 35.7 against 41.0
        // us at 4096 blobs, 41.3 and 41.7 at 4480 (43.7 and 41.9 at 4608).
        const bool third = items > 512 && items <= 640;
        s.ok = s.ok && prec == RPYW_FP64 && N <= (K == 1 ? kSym2MaxN1 : kSym2MaxN) &&
               (K > 1 || (N >= kSym2MinN1 && !third));
    }
    return s;
}

SymPlan sym_choose(int64_t N, int prec, int K, const Shape& sh, const Domain& dom) {
    if (prec == RPYW_FP64 && !dom.periodic()) {
        const SymPlan s = sym_plan(N, prec, K, sh.ipw2 ? sh.ipw2 : sh.ipw, 128);
        if (s.ok || K > 1) return s;
    }
    // Periodic products are always symmetric: groups of 64 unless the shape
    // asks for groups of 256.
    const bool g64 = dom.periodic() ? sh.sym != 1 : sh.sym == 2;
    if (g64) {
        const SymPlan s = sym_plan(N, prec, K, sh.ipw, 64);
        if (s.ok) return s;
    }
    return sym_plan(N, prec, K, sh.ipw, 256);
}

void split_plan(int64_t N, int tpl, int* splits, int64_t* chunk) {
    const int64_t ntb = (N + (int64_t)kBlock * tpl - 1) / ((int64_t)kBlock * tpl);
    const int64_t want_wg = 2048;
    int64_t s = (want_wg + ntb - 1) / ntb;
    const int64_t max_s = std::max<int64_t>(1, N / 64);
    if (s > max_s) s = max_s;
    if (s > 8) s = (s + 7) / 8 * 8;
    if (s < 1) s = 1;
    int64_t c = (N + s - 1) / s;
    s = (N + c - 1) / c;
    *splits = (int)s;
    *chunk = c;
}

// Source chunks of the matrix-core kernel: workgroups of 64 targets, enough
// of them for several rounds of five per CU (the tail of the last round
// then costs little), chunks of at least 256 sources.
// Chunks are shared out at multiples of the LDS tile while that makes kMatWgs
// workgroups or fewer (as many as run at a time): until then the kernel is bound
// by the chain of a wave's steps, 0.7 us for 4 sources.  FP32C, 16 right-hand
// sides, a call: 300 blobs 53.9 -> 29.5 us, 1000 blobs 59.1 -> 31.0; sharing
// further lost at 3000 (68 -> 77).
constexpr int64_t kMatWgs = 1280;
MatSplit mat_split_plan(int64_t N, int prec) {
    const int64_t ntb = (N + kMatTargets - 1) / kMatTargets;
    const int64_t want_wg = 8192;
    int64_t s = (want_wg + ntb - 1) / ntb;
    const int64_t max_s = std::max<int64_t>(1, N / 256);
    if (s > max_s) s = max_s;
    if (s > 8) s = (s + 7) / 8 * 8;
    if (s < 1) s = 1;
    MatSplit m;
    m.chunk = (N + s - 1) / s;
    s = (N + m.chunk - 1) / m.chunk;
    const int tile = prec == RPYW_FP32C ? mat_tile<float>() : mat_tile<double>();
    const int64_t tiles = (m.chunk + tile - 1) / tile;
    const int64_t fit = std::max<int64_t>(1, std::min<int64_t>(tiles, kMatWgs / (ntb * s)));
    m.sublen = (int)((tiles + fit - 1) / fit) * tile;
    m.sub = (int)((m.chunk + m.sublen - 1) / m.sublen);
    m.splits = (int)s * m.sub;
    return m;
}

size_t product_ws_bytes(int64_t N, int prec, int kblk) {
    int s1, s2, s3 = 1;
    int64_t c;
    split_plan(N, 1, &s1, &c);
    split_plan(N, 2, &s2, &c);
    if (kblk >= 8) s3 = mat_split_plan(N, prec).splits;
    const int smax = std::max(std::max(s1, s2), s3);
    size_t b = align_up((size_t)N * rec_width(prec, kblk) * real_size(prec));
    b += align_up((size_t)N * sizeof(double));
    b += align_up((size_t)smax * kblk * 3 * N * sizeof(double));
    size_t sb = 0;
    for (int K = 1; K <= std::min(kblk, 4); K <<= 1)
        for (int G : {256, 128, 64}) {
            // FP64 blocks of two and four have only groups of 128, and two
            // right-hand sides of a periodic product groups of 64
            if (prec == RPYW_FP64 && ((K > 1 && G == 256) || (K > 2 && G == 64))) continue;
            // one item to a workgroup has the most partials; where these are too
            // many for the kernel, two (FP32C, whose source partials are floats;
            // of wider blocks, which only a fixed shape has, those that do not
            // fit go to the plain kernel)
            SymPlan sp = sym_plan(N, prec, K, 1, G);
            if (!sp.ok && K == 1) sp = sym_plan(N, prec, K, 2, G);
            if (sp.ok) sb = std::max(sb, sp.rec_bytes + sp.tpart_bytes + sp.spart_bytes);
        }
    return std::max(b, sb) + 8 * kAlign;
}

namespace {

int sym_pass(const double* pos, const double* F, double* U, int64_t N, int kb, int K, double a, double eta, int prec,
             const SymPlan& sp, Arena& ar, hipStream_t st, const Domain& dom = Domain{}) {
    const size_t mark = ar.used;
    double* tpart = (double*)ar.take(sp.tpart_bytes);
    void* spart = ar.take(sp.spart_bytes);
    if (!tpart || !spart) {
        ar.used = mark;
        return RPYW_ENOMEM;
    }
    // Groups of 64 and of 128: the pair kernel forms the records itself, two
    // launches per product; otherwise the records are packed once by their
    // own kernel.  So are those of FP32C products in a periodic cell whose
    // passes are not split: forming them there is a wrap in FP64 per record,
    // and the kernel that reads them needs 94 vector registers instead of 106
    // (5 waves on a SIMD, not 4): 2.53 -> 2.46 ms at 20000 blobs, 5.64 -> 5.49
    // at 29958.  In FP64 the packed form is the slower one (two right-hand
    // sides at 20000 blobs: 5.73 ms, formed in the kernel 5.49).
    const bool fused = sp.G != 256 && !(dom.periodic() && prec == RPYW_FP32C && sp.ns == 1);
    const PackSrc ps{pos, F, N, kb, 1.0 / a, dom.lx / a, dom.ly / a};
    void* rec = nullptr;
    double* B = nullptr;
    int rc = RPYW_OK;
    if (!fused) {
        const int rw = rec_width(prec, K);
        const int64_t npad = (int64_t)sp.ng * sp.G;
        rec = ar.take((size_t)npad * rw * real_size(prec));
        B = (double*)ar.take((size_t)npad * sizeof(double));
        if (!rec || !B) {
            ar.used = mark;
            return RPYW_ENOMEM;
        }
        rc = sym_pack(pos, F, N, kb, K, prec, sp, a, dom, rec, B, st);
    }
    if (rc == RPYW_OK) {
        hipEvent_t ev = nullptr;
        profile_begin(st, &ev);
        rc = sym_launch(rec, sp, K, prec, a, dom, tpart, spart, st, fused ? &ps : nullptr);
        if (rc == RPYW_OK) {
            profile_end(st, ev, (dom.periodic() ? 9.0 : 1.0) * (double)kb * (double)N * (double)N);
            rc = sym_finish(tpart, spart, B, N, kb, K, prec, sp, mu0_of(a, eta), U, st, pos, 1.0 / a);
        }
    }
    ar.used = mark;
    return rc;
}

}  // namespace

int sym_pack(const double* pos, const double* F, int64_t N, int kb, int K, int prec, const SymPlan& sp, double a,
             const Domain& dom, void* rec, double* B, hipStream_t st) {
    const int rw = rec_width(prec, K);
    const int64_t npad = (int64_t)sp.ng * sp.G;
    const unsigned g1 = (unsigned)((npad + kBlock - 1) / kBlock);
    if (prec == RPYW_FP32C)
        hipLaunchKernelGGL(pack_kernel<float>, dim3(g1), dim3(kBlock), 0, st, pos, F, N, kb, rw, 1.0 / a, (float*)rec, B,
                           nullptr, dom.lx / a, dom.ly / a, npad);
    else
        hipLaunchKernelGGL(pack_kernel<double>, dim3(g1), dim3(kBlock), 0, st, pos, F, N, kb, rw, 1.0 / a,
                           (double*)rec, B, nullptr, dom.lx / a, dom.ly / a, npad);
    RPYW_HIP(hipGetLastError());
    return RPYW_OK;
}

int sym_launch(const void* rec, const SymPlan& sp, int K, int prec, double a, const Domain& dom, double* tpart,
               void* spart, hipStream_t st, const PackSrc* ps) {
    auto go = [&](auto Rt, auto Kc) -> hipError_t {
        using R = decltype(Rt);
        constexpr int KK = decltype(Kc)::value;
        if (dom.periodic()) {
            if constexpr (KK <= 2) {
                // FP64 only: in FP32 the branch-free far images measured
                // 4-7% slower, in FP64 up to 10% faster
                if constexpr (sizeof(R) == 8)
                    if (std::min(dom.lx, dom.ly) > 4.5 * a)
                        return launch_sym_t<R, KK, 2>((const R*)rec, sp, tpart, (R*)spart, make_box<R>(dom, a), st, ps);
                return launch_sym_t<R, KK, 1>((const R*)rec, sp, tpart, (R*)spart, make_box<R>(dom, a), st, ps);
            }
            return hipErrorInvalidValue;
        }
        if constexpr (sizeof(R) == 8)
            if (sp.G == 128) return launch_sym2_t<KK>((const R*)rec, sp, tpart, (R*)spart, st, ps);
        if constexpr (sizeof(R) == 4 || KK == 1)  // FP64 has the other groups for one right-hand side
            return launch_sym_t<R, KK, 0>((const R*)rec, sp, tpart, (R*)spart, Box<R>{}, st, ps);
        return hipErrorInvalidValue;
    };
    hipError_t e;
    if (prec == RPYW_FP32C)
        e = K == 1 ? go(0.f, std::integral_constant<int, 1>{})
                   : K == 2 ? go(0.f, std::integral_constant<int, 2>{}) : go(0.f, std::integral_constant<int, 4>{});
    else
        e = K == 1 ? go(0.0, std::integral_constant<int, 1>{})
                   : K == 2 ? go(0.0, std::integral_constant<int, 2>{}) : go(0.0, std::integral_constant<int, 4>{});
    return e == hipSuccess ? RPYW_OK : RPYW_EHIP;
}

int sym_finish(const double* tpart, const void* spart, const double* B, int64_t N, int kb, int K, int prec,
               const SymPlan& sp, double mu0, double* U, hipStream_t st, const double* pos, double inv_a) {
    if (!B && !pos) return RPYW_EINVAL;
    const dim3 ge((unsigned)((N + 63) / 64), (unsigned)(3 * kb));
    if (prec == RPYW_FP32C)
        hipLaunchKernelGGL(sym_epilogue<float>, ge, dim3(64 * kEpiParts), 0, st, tpart, (const float*)spart, B, N,
                           sp.ng, sp.C, sp.Hmax, sp.nseg, K, sp.G, mu0, U, pos, inv_a);
    else
        hipLaunchKernelGGL(sym_epilogue<double>, ge, dim3(64 * kEpiParts), 0, st, tpart, (const double*)spart, B, N,
                           sp.ng, sp.C, sp.Hmax, sp.nseg, K, sp.G, mu0, U, pos, inv_a);
    RPYW_HIP(hipGetLastError());
    return RPYW_OK;
}

int product_pass(const double* pos, const double* F, double* U, int64_t N, int kb, double a, double eta, int prec,
                 Shape sh, Arena& ar, hipStream_t st) {
    const size_t mark = ar.used;
    const int K = kernel_k(kb, prec, sh.mat);
    if (kb < 1 || kb > K) return RPYW_EINVAL;
    sh = normalized(sh, K, prec);
    if (sh.sym && K <= 4) {
        const SymPlan sp = sym_choose(N, prec, K, sh, Domain{});
        if (sp.ok) {
            const int rc = sym_pass(pos, F, U, N, kb, K, a, eta, prec, sp, ar, st);
            if (rc != RPYW_ENOMEM) return rc;
        }
    }
    const int rw = rec_width(prec, K);
    void* rec = ar.take((size_t)N * rw * real_size(prec));
    double* B = (double*)ar.take((size_t)N * sizeof(double));
    int splits;
    int64_t chunk;
    MatSplit ms{};
    if (sh.mat) {
        ms = mat_split_plan(N, prec);
        splits = ms.splits;
    } else {
        split_plan(N, sh.tpl, &splits, &chunk);
    }
    double* part = (double*)ar.take((size_t)splits * K * 3 * N * sizeof(double));
    if (!rec || !B || !part) {
        ar.used = mark;
        return RPYW_ENOMEM;
    }
    RPYW_HIP(launch_pack(prec, K, pos, F, N, kb, a, rec, B, st));
    const int span = sh.mat ? kMatTargets : kBlock * sh.tpl;
    const int64_t ntb = (N + span - 1) / span;
    const int64_t nblocks = ntb * splits;
    hipEvent_t ev = nullptr;
    profile_begin(st, &ev);
    hipError_t e;
    if (sh.mat)
        e = launch_mat(prec, K, rec, N, ms, part, nblocks, st);
    else if (prec == RPYW_FP32C)
        e = RPYW_DISPATCH(float, K, sh.tpl, sh.tile, launch_pair_t, (const float*)rec, N, splits, chunk, part, nblocks,
                          st);
    else
        e = RPYW_DISPATCH(double, K, sh.tpl, sh.tile, launch_pair_t, (const double*)rec, N, splits, chunk, part,
                          nblocks, st);
    if (e != hipSuccess) return RPYW_EHIP;
    profile_end(st, ev, (double)kb * (double)N * (double)N);
    hipLaunchKernelGGL(epilogue_kernel, dim3((unsigned)((N + 63) / 64), (unsigned)(3 * kb)), dim3(64 * kEpiParts), 0, st,
                       part, B, N, K, splits, mu0_of(a, eta), U);
    RPYW_HIP(hipGetLastError());
    ar.used = mark;
    return RPYW_OK;
}

namespace {

// FP64 products of small problems, in blocks of up to 8 right-hand sides.
template <int K>
void launch_direct(const double* pos, const double* F, double* U, int64_t N, int kb, double a, double eta,
                   hipStream_t st) {
    hipLaunchKernelGGL((direct_kernel<K>), dim3((unsigned)((N + kDirectTargets - 1) / kDirectTargets)),
                       dim3(kDirectThreads), 0, st, pos, F, N, kb, 1.0 / a, mu0_of(a, eta), U);
}

int direct_products(const double* pos, const double* F, double* U, int64_t N, int k, double a, double eta,
                    hipStream_t st) {
    for (int k0 = 0; k0 < k; k0 += 8) {
        const int kb = std::min(8, k - k0);
        const double* Fk = F + (size_t)k0 * N * 3;
        double* Uk = U + (size_t)k0 * N * 3;
        hipEvent_t ev = nullptr;
        profile_begin(st, &ev);
        if (kb == 1)
            launch_direct<1>(pos, Fk, Uk, N, kb, a, eta, st);
        else if (kb == 2)
            launch_direct<2>(pos, Fk, Uk, N, kb, a, eta, st);
        else if (kb <= 4)
            launch_direct<4>(pos, Fk, Uk, N, kb, a, eta, st);
        else
            launch_direct<8>(pos, Fk, Uk, N, kb, a, eta, st);
        RPYW_HIP(hipGetLastError());
        profile_end(st, ev, (double)kb * (double)N * (double)N);
    }
    return RPYW_OK;
}

bool overlap(const double* x, int64_t nx, const double* y, int64_t ny) {
    const uintptr_t a = (uintptr_t)x, b = (uintptr_t)y;
    return a < b + (size_t)ny * sizeof(double) && b < a + (size_t)nx * sizeof(double);
}

}  // namespace

int products(const double* pos, const double* F, double* U, int64_t N, int k, double a, double eta, int prec,
             Arena& ar, hipStream_t st, const Domain& dom) {
    if (dom.periodic()) {
        // Always symmetric.  Over groups of 64 right-hand sides go two to a pass
        // (the nine images' coefficients are most of the work), with the sums of
        // single passes, if the workspace holds the partials of two.  A call with
        // two, FP32C and FP64: 1202 blobs 39.6 -> 25.3 and 50.7 -> 33.6 us, 20000
        // blobs 5.10 -> 3.52 and 9.2 -> 5.8 ms.
        const Shape sh = tuned_shape(N, 1, prec);
        const SymPlan sp = sym_choose(N, prec, 1, sh, dom);
        if (!sp.ok) return RPYW_ENOMEM;
        const SymPlan sp2 = sym_choose(N, prec, 2, sh, dom);
        bool two = sp2.ok && sp2.G == 64 && sp.G == 64;
        for (int k0 = 0; k0 < k;) {
            const double* Fk = F + (size_t)k0 * N * 3;
            double* Uk = U + (size_t)k0 * N * 3;
            const int kb = two && k - k0 >= 2 ? 2 : 1;
            const int rc = sym_pass(pos, Fk, Uk, N, kb, kb, a, eta, prec, kb == 2 ? sp2 : sp, ar, st, dom);
            if (rc == RPYW_ENOMEM && kb == 2) {
                two = false;
                continue;
            }
            if (rc != RPYW_OK) return rc;
            k0 += kb;
        }
        return RPYW_OK;
    }
    return shaped_products(pos, F, U, N, k, a, eta, prec, tuned_shape(N, k, prec), ar, st);
}

int shaped_products(const double* pos, const double* F, double* U, int64_t N, int k, double a, double eta, int prec,
                    Shape sh, Arena& ar, hipStream_t st) {
    // One launch writes velocities while other workgroups still read: outputs
    // on top of the inputs take the other kernels, which read them all first.
    if (sh.direct && !overlap(U, 3 * N * k, F, 3 * N * k) && !overlap(U, 3 * N * k, pos, 3 * N))
        return direct_products(pos, F, U, N, k, a, eta, st);
    if (prec != RPYW_FP32C && !sh.mat) sh.kblk = std::min(sh.kblk, 8);  // e.g. RPYW_RHS_WIDTH=16 on the vector units
    for (int k0 = 0; k0 < k; k0 += sh.kblk) {
        const int kb = std::min(sh.kblk, k - k0);
        const int rc = product_pass(pos, F + (size_t)k0 * N * 3, U + (size_t)k0 * N * 3, N, kb, a, eta, prec, sh, ar,
                                    st);
        if (rc != RPYW_OK) return rc;
    }
    return RPYW_OK;
}

// ------------------------------------------------------------ batched

size_t batched_ws_bytes(int64_t Ntot, int S, int k, int prec, bool split) {
    const int kb = kernel_k(std::max(k, 1), prec, 1);  // the widest the batched kernels take
    size_t b = align_up((size_t)Ntot * rec_width(prec, kb) * real_size(prec));
    b += align_up((size_t)Ntot * sizeof(double));
    size_t items = (size_t)(Ntot / kMatTargets) + (size_t)S + 1;  // items of 64 or more targets
    if (split) {
        const bool mat = default_shape(Ntot, std::max(k, 1), prec).mat;
        const int parts = batched_parts(Ntot / (mat ? kMatTargets : kBlock) + 1, mat);
        if (parts > 1) {
            items += kBatchedItems;
            b += align_up((size_t)parts * kernel_k(std::max(k, 1), prec, mat) * 3 * Ntot * sizeof(double));
            b += align_up((size_t)Ntot * sizeof(int));
        }
    }
    b += align_up(items * sizeof(int4));
    b += kAlign;  // counter
    return b + 4 * kAlign;
}

int batched_products(const double* pos, const int64_t* sys_offsets, int S, const double* F, double* U, int k,
                     double a, double eta, int prec, Arena& ar, hipStream_t st) {
    const int64_t Ntot = sys_offsets[S];
    int64_t nmax = 0;
    for (int s = 0; s < S; ++s) nmax = std::max(nmax, sys_offsets[s + 1] - sys_offsets[s]);
    // The batched kernel is the plain one, with the widest RHS block (one
    // pass over the sources per item): the shapes tuned for products of one
    // system (a symmetric kernel, or narrower blocks that fill the GPU with a
    // single system) do not carry over to a persistent launch over many; the
    // RPYW_TILE / RPYW_RHS_WIDTH overrides still apply.
    Shape sh = default_shape(nmax, k, prec);
    sh.sym = 0;
    sh.kblk = widest_block(k, prec);
    sh = apply_env_overrides(sh);
    sh = normalized(sh, kernel_k(sh.kblk, prec, sh.mat), prec);
    const int span = sh.mat ? kMatTargets : kBlock * sh.tpl;
    const int tile = !sh.mat ? (sh.tile == 64 ? 64 : 256)
                     : prec == RPYW_FP32C ? mat_tile<float>() : mat_tile<double>();
    const size_t mark = ar.used;
    const int K = kernel_k(sh.kblk, prec, sh.mat);
    if (sh.kblk > K) return RPYW_EINVAL;
    const int rw = rec_width(prec, K);
    void* rec = ar.take((size_t)Ntot * rw * real_size(prec));
    double* B = (double*)ar.take((size_t)Ntot * sizeof(double));
    unsigned* counter = (unsigned*)ar.take(sizeof(unsigned));
    // items with one part (more than kBatchedItems systems are never split)
    int64_t whole = std::max<int64_t>(Ntot / (sh.mat ? kMatTargets : kBlock) + 1, S);
    if (S < kBatchedItems) {
        int64_t n = 0;
        for (int s = 0; s < S; ++s) n += (sys_offsets[s + 1] - sys_offsets[s] + span - 1) / span;
        whole = std::max(whole, n);
    }
    // the sources in one part if the workspace does not hold more
    int parts = batched_parts(whole, sh.mat);
    const int64_t from = split_from(whole, sh.mat, nmax, span);
    std::vector<BatchedItem> items;
    static_assert(sizeof(BatchedItem) == sizeof(int4));
    int4* ditems = nullptr;
    double* part = nullptr;
    int* used = nullptr;
    for (const size_t before = ar.used;; parts = 1) {
        ar.used = before;
        parts = batched_items(sys_offsets, S, span, tile, parts, from, whole, items);
        ditems = (int4*)ar.take(items.size() * sizeof(int4));
        if (parts == 1) break;
        part = (double*)ar.take((size_t)parts * K * 3 * Ntot * sizeof(double));
        used = (int*)ar.take((size_t)Ntot * sizeof(int));
        if (ditems && part && used) break;
        part = nullptr;
    }
    if (!rec || !B || !ditems || !counter) {
        ar.used = mark;
        return RPYW_ENOMEM;
    }
    int rc = stage_upload(items.data(), items.size() * sizeof(int4), ditems, st);
    if (rc != RPYW_OK) return rc;
    int dev = 0, ncu = 256;
    RPYW_HIP(hipGetDevice(&dev));
    RPYW_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    const int per_cu = sh.mat ? (prec == RPYW_FP32C ? mat_batched_waves<float>() : mat_batched_waves<double>()) : 4;
    const int grid = (int)std::min<size_t>(items.size(), (size_t)ncu * per_cu);
    const double m0 = mu0_of(a, eta);
    double pairs = 0.0;
    for (int s = 0; s < S; ++s) {
        const double n = (double)(sys_offsets[s + 1] - sys_offsets[s]);
        pairs += n * n;
    }
    for (int k0 = 0; k0 < k; k0 += sh.kblk) {
        const int kb = std::min(sh.kblk, k - k0);
        const double* Fk = F + (size_t)k0 * Ntot * 3;
        double* Uk = U + (size_t)k0 * Ntot * 3;
        RPYW_HIP(launch_pack(prec, K, pos, Fk, Ntot, kb, a, rec, B, st));
        hipLaunchKernelGGL(zero_u32, dim3(1), dim3(1), 0, st, counter);
        RPYW_HIP(hipGetLastError());
        hipEvent_t ev = nullptr;
        profile_begin(st, &ev);
        hipError_t e;
        if (sh.mat)
            e = launch_mat_batched(prec, K, rec, ditems, (int)items.size(), counter, B, m0, Ntot, kb, Uk, part, used,
                                   grid, st);
        else if (prec == RPYW_FP32C)
            e = RPYW_DISPATCH(float, K, sh.tpl, sh.tile, launch_batched_t, (const float*)rec, ditems,
                              (int)items.size(), counter, B, m0, Ntot, kb, Uk, part, used,
                                   grid, st);
        else
            e = RPYW_DISPATCH(double, K, sh.tpl, sh.tile, launch_batched_t, (const double*)rec, ditems,
                              (int)items.size(), counter, B, m0, Ntot, kb, Uk, part, used,
                                   grid, st);
        if (e != hipSuccess) return RPYW_EHIP;
        profile_end(st, ev, kb * pairs);
        if (parts > 1) {
            hipLaunchKernelGGL(epilogue_kernel, dim3((unsigned)((Ntot + 63) / 64), (unsigned)(3 * kb)),
                               dim3(64 * kEpiParts), 0, st, part, B, Ntot, K, parts, m0, Uk, used);
            RPYW_HIP(hipGetLastError());
        }
    }
    ar.used = mark;
    return RPYW_OK;
}

}  // namespace rpyw
