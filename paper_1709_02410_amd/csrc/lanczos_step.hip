// Fused steps of the preconditioned Lanczos iteration for M^{1/2} W
// (arXiv:1709.02410, Sec. II.B) when the product runs through the symmetric
// pair kernel.  Step k is four launches:
//   vin   one workgroup per body (per 21 blobs without bodies): the second
//         Gram-Schmidt correction and normalisation of the previous step,
//         v_k = (y' - V c2) / beta_{k-1}, with c2 = V^T y' and |y'|^2 added
//         up from the block partials of gs2 in a fixed order (every
//         workgroup repeats that small sum); then x = L^-T v_k, written
//         straight into the force slots of the pair kernel's records
//         (B x in the kernel precision; the positions are packed once);
//   pair  the symmetric pair kernel: M x as partial sums;
//   out   one workgroup per group of whole bodies (at most 64 entries, or
//         one larger body): y = M x gathered from the partial sums (eight
//         or four threads per entry, fixed order), w = L^-1 y -
//         beta_{k-1} v_{k-1} (the inverse factors staged through LDS), and
//         the group's partial dot products V_j . w (j <= k), one wave per
//         vector;
//   gs2   blocks of consecutive entries: c1 = V^T w added up from the
//         partials of out, alpha_k = c1[k], y' = w - V c1 (the first
//         correction), and the block partials of V^T y' and |y'|^2.
// The first correction and the second projection are the two classical
// Gram-Schmidt passes of the full reorthogonalisation; beta_k =
// (|y'|^2 - |c2|^2)^{1/2} as in the unfused driver.  vin of step k + 1 is
// launched with step k: its first workgroup publishes step k (alpha_k, kept
// in device memory by gs2, and beta_k) into pinned memory, where the host
// polls them.
#include <algorithm>
#include <cmath>
#include <vector>

#include "krylov_step.h"
#include "records.h"
#include "rpyw_internal.h"
#include "sym_pairs.h"

namespace rpyw {

namespace {

using namespace kstep;

constexpr int kVinThreads = 256;
constexpr int kOutThreads = 512;
constexpr int kGs2Threads = 256;
constexpr int kVinReg = 16;  // basis values a thread of vin keeps in registers
constexpr int kPackThreads = 256;

// vin and out are chains of dependent round trips (loads, the sums over them,
// the factor) on one workgroup per body, and are bound by the length of the
// chain: the loads go out first, with the partials that start the chain ahead
// of the others; several threads share an entry's sums over the basis and the
// rows of the factor; the norm is a wave's sum.  One thread per entry took 7.6
// us (vin) and 8.9 us (out) a step on 256 boomerangs, now 5.9 and 6.9.
template <typename R>
__global__ __launch_bounds__(kVinThreads) void lz_vin_kernel(int diag, const int* __restrict__ units,
                                                             const int64_t* __restrict__ lofs,
                                                             const double* __restrict__ Lall, int64_t n3, int k,
                                                             const double* __restrict__ src,
                                                             const double* __restrict__ part2, int ncol2,
                                                             double* __restrict__ V, double* __restrict__ d_ab,
                                                             double* __restrict__ h_ab,
                                                             R* __restrict__ rec, int recw,
                                                             const double* __restrict__ B,
                                                             double* __restrict__ h_hdr,
                                                             const int* __restrict__ bad0,
                                                             const int* __restrict__ bad1) {
    constexpr int PW = pos_slots<R>();
    __shared__ double c[kLanczosFusedMaxIter + 2];
    __shared__ double x[3 * kMaxBodyBlobs];
    __shared__ double Li[kLdsFactor];
    __shared__ double upd[kVinThreads];
    __shared__ double sinv;
    const int p = blockIdx.x, t = threadIdx.x;
    // the partials of gs2 first (they depend on nothing this kernel loads; at
    // k = 0 the packing kernel's partials of |W|^2)
    RowSums<kVinThreads> rows;
    rows.load(part2, k + 1, ncol2);
    const int64_t e0 = 3 * (int64_t)units[p];
    const int n = (int)(3 * (int64_t)units[p + 1] - e0);
    const bool lds_factor = !diag && n * n <= kLdsFactor;
    // Units of up to 64 entries: four threads per entry (quarter t / 64), which
    // take the vectors j = quarter (mod 4); larger ones (up to 126): two.
    const int ways = n <= 64 ? 4 : 2, el = n <= 64 ? t & 63 : t & 127, qr = wave_uniform(n <= 64 ? t >> 6 : t >> 7);
    // loads that do not depend on the reductions go next: the inverse factor,
    // this entry's source value, B of its blob and its basis values
    Staged<kVinThreads, kLdsFactor / kVinThreads> sf;
    if (lds_factor) sf.load(Lall + 2 * lofs[p] + (int64_t)n * n, n * n);
    const bool has = el < n;
    const int64_t ec = e0 + (has ? el : 0);  // an in-bounds address for idle lanes
    // entry of the record that this thread writes: four lanes apply the factor
    // of each entry when the entries allow it
    const bool spread = lds_factor && n <= 64;
    const int ei = spread ? t >> 2 : t;
    double vr = t < n ? src[e0 + t] : 0.0;
    const double bb = ei < n ? B[(e0 + ei) / 3] : 0.0;
    const double alpha = p == 0 && t == 0 && k > 0 ? d_ab[2 * (k - 1)] : 0.0;
    double a[kVinReg];
#pragma unroll
    for (int i0 = 0; i0 < kVinReg; i0 += 4) {
        if (ways * i0 >= k) break;  // uniform
#pragma unroll
        for (int i = i0; i < i0 + 4; ++i) {
            const int j = qr + ways * i;
            a[i] = V[(j < k ? j : 0) * n3 + ec];
        }
    }
    rows.finish(part2, k + 1, ncol2, c);  // c[0..k) = c2, c[k] = |y'|^2 (k = 0: |W|^2)
    // the second correction, and by the first wave the norm
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < kVinReg; ++i)
        if (qr + ways * i < k) s = fma(c[qr + ways * i], a[i], s);
    for (int j = qr + ways * kVinReg; j < k; j += ways) s = fma(c[j], V[j * n3 + ec], s);
    upd[t] = s;
    if (t < 64) {
        double q = 0.0;
        for (int j = t; j < k; j += 64) q = fma(c[j], c[j], q);
        const double s2 = c[k] - lane_group_sum<64>(q);
        const double b = s2 > 0.0 ? sqrt(s2) : 0.0;
        if (t == 0) {
            sinv = 1.0 / b;  // b = 0: breakdown, this step's values are discarded
            if (p == 0 && k > 0) {
                // publish step k - 1: alpha (kept by its gs2) and beta
                d_ab[2 * (k - 1) + 1] = b;
                publish(h_ab + 2 * (k - 1), alpha);
                publish(h_ab + 2 * (k - 1) + 1, b);
            } else if (p == 0) {
                publish_header(h_hdr, b, bad0, bad1);  // beta_0 = |W|
            }
        }
    }
    if (lds_factor) sf.store(Li, n * n);  // read after the next barrier
    __syncthreads();
    if (t < n) {
        const double v = (vr - (ways == 4 ? (upd[t] + upd[t + 64]) + (upd[t + 128] + upd[t + 192])
                                          : upd[t] + upd[t + 128])) *
                         sinv;
        V[k * n3 + e0 + t] = v;
        x[t] = v;
    }
    __syncthreads();
    // x <- (L_p^-1)^T x, row e: column e of L_p^-1 from its diagonal down
    if (ei < n) {
        double z;
        if (spread) {
            z = 0.0;
            for (int m = ei + (t & 3); m < n; m += 4) z = fma(Li[m * n + ei], x[m], z);
            z = lane_group_sum<4>(z);
        } else {
            z = diag         ? x[t] / Lall[e0 + t]
                : lds_factor ? dot4(Li + t * n + t, n, x + t, n - t)
                             : dot4(Lall + 2 * lofs[p] + (int64_t)n * n + t * n + t, n, x + t, n - t);
        }
        const int64_t blob = (e0 + ei) / 3;
        if (!spread || (t & 3) == 0) rec[blob * recw + PW + (int)(e0 + ei - 3 * blob)] = (R)(bb * z);
    }
}

template <typename R>
__global__ __launch_bounds__(kOutThreads) void lz_out_kernel(
    int diag, const int* __restrict__ units, const LanczosGroup* __restrict__ ginfo,
    const double* __restrict__ Lall, const double* __restrict__ tpart, const R* __restrict__ spart, int ng, int C,
    int Hmax, int nseg, int G, const double* __restrict__ B, double mu0, int64_t n3, int k,
    const double* __restrict__ V, const double* __restrict__ d_ab, double* __restrict__ w,
    double* __restrict__ part1, int ngroups, const double* __restrict__ ypre) {
    __shared__ double red[kOutThreads];
    __shared__ double y[3 * kMaxBodyBlobs];  // a group has at most 64 entries, or one body of up to 126
    __shared__ double wl[3 * kMaxBodyBlobs];
    __shared__ double Lf[2 * kLdsFactor];    // the group's factors as stored: L_p, then L_p^-1, per body
    __shared__ int ub[kLanczosGroupUnits + 1];
    const int g = blockIdx.x, t = threadIdx.x;
    // everything that does not depend on the product goes first: the group
    // (one table entry), then its unit offsets, factors, B, the previous
    // basis vector and beta_{k-1}, and the basis values of the dot products
    const LanczosGroup gi = ginfo[g];
    const int g0 = gi.g0, nu = gi.g1 - gi.g0;
    const int64_t e0 = 3 * (int64_t)gi.b0;
    const int n = 3 * (gi.b1 - gi.b0);
    // threads per entry: 8 for groups of up to 64 entries, 4 up to 128
    const int U = n <= 64 ? 8 : 4;
    const bool lds_factor = !diag && gi.sq <= kLdsFactor;
    const int uv = t <= nu ? units[g0 + t] : 0;
    Staged<kOutThreads, 2 * kLdsFactor / kOutThreads> sf;
    if (lds_factor) sf.load(Lall + 2 * gi.loff, 2 * gi.sq);
    // the factor of a group of up to 64 entries is applied by eight lanes per
    // entry (entry t / 8), otherwise by thread t for entry t
    const bool spread = lds_factor && n <= 64;
    const int et = spread ? t >> 3 : t;
    const bool has = et < n && (!spread || (t & 7) == 0);
    double vprev = 0.0, bb = 0.0, dg = 0.0;
    if (has && k > 0) vprev = V[(k - 1) * n3 + e0 + et];
    if (t < n) {
        bb = B[(e0 + t) / 3];
        if (diag) dg = Lall[e0 + t];
    }
    const double bk = k > 0 ? d_ab[2 * (k - 1) + 1] : 0.0;
    // the lane's basis values for the dot products (waves take the vectors
    // j = wave (mod 8), lanes the entries l and l + 64), loaded ahead
    const int wv = wave_uniform(t >> 6), l = t & 63;
    constexpr int kWaves = kOutThreads / 64;
    double av[kWaves][2];
#pragma unroll
    for (int i = 0; i < kWaves; ++i) {
        const int j = wv + kWaves * i;
        av[i][0] = (j <= k && l < n) ? V[j * n3 + e0 + l] : 0.0;
        av[i][1] = (j <= k && l + 64 < n) ? V[j * n3 + e0 + l + 64] : 0.0;
    }
    const int S = gather_slots(n);  // U = kOutThreads / S
    if (!ypre) {
        const int slot = t % S, u = t / S;
        double r = 0.0;
        if (slot < n) {
            const int64_t e = e0 + gather_entry(slot, n), blob = e / 3;
            r = gather_share<R>(tpart, spart, blob, ng, C, Hmax, nseg, G, (int)(e - 3 * blob), u, U);
        }
        red[t] = r;
    }
    if (t <= nu) ub[t] = uv;
    if (lds_factor) sf.store(Lf, 2 * gi.sq);
    __syncthreads();
    if (t < n && ypre) {
        y[t] = ypre[e0 + t];
    } else if (t < n) {
        const double* rt = red + gather_slot(t, n);
        double s = rt[0];
        if (U == 8) {
#pragma unroll
            for (int u = 1; u < 8; ++u) s += rt[u * 64];
        } else {
#pragma unroll
            for (int u = 1; u < 4; ++u) s += rt[u * 128];
        }
        y[t] = mu0 * bb * s;
    }
    __syncthreads();
    if (et < n) {
        double v;
        if (diag) {
            v = y[t] / dg;
        } else {
            // the entry's body (unit offsets in LDS) and where its factors
            // start relative to the group's
            int q = 0, off = 0;
            while (3 * (ub[q + 1] - ub[0]) <= et) {
                const int nq = 3 * (ub[q + 1] - ub[q]);
                off += 2 * nq * nq;
                ++q;
            }
            const int bs = 3 * (ub[q] - ub[0]), bn = 3 * (ub[q + 1] - ub[q]);
            const int i = et - bs;
            const int64_t fi = off + (int64_t)bn * bn + (int64_t)i * bn;  // row i of L_p^-1
            if (spread) {
                v = 0.0;
                for (int m = t & 7; m <= i; m += 8) v = fma(Lf[fi + m], y[bs + m], v);
                v = lane_group_sum<8>(v);
            } else {
                v = lds_factor ? dot4(Lf + fi, 1, y + bs, i + 1) : dot4(Lall + 2 * gi.loff + fi, 1, y + bs, i + 1);
            }
        }
        if (has) {
            if (k > 0) v -= bk * vprev;
            w[e0 + et] = v;
            wl[et] = v;
        }
    }
    __syncthreads();
    const double w0 = l < n ? wl[l] : 0.0, w1 = l + 64 < n ? wl[l + 64] : 0.0;
    {
        // the wave's kWaves dot products folded together
        double pr[kWaves];
#pragma unroll
        for (int i = 0; i < kWaves; ++i) pr[i] = fma(av[i][1], w1, fma(av[i][0], w0, 0.0));
        wave_fold<kWaves, 32>(pr);
        const int j = wv + kWaves * wave_value<kWaves>(l);
        if (l % (64 / kWaves) == 0 && j <= k) part1[(int64_t)j * ngroups + g] = pr[0];
    }
    for (int j = wv + kWaves * kWaves; j <= k; j += kWaves) {
        const double* Vj = V + j * n3 + e0;
        double p = fma(l < n ? Vj[l] : 0.0, w0, 0.0);
        p = fma(l + 64 < n ? Vj[l + 64] : 0.0, w1, p);
        p = lane_group_sum<64>(p);
        if (l == 0) part1[(int64_t)j * ngroups + g] = p;
    }
}

// gs2: c1 from the partials of out; y' = w - sum_{j <= k} c1[j] V_j, and block
// partials of V_j . y' (j <= k) and |y'|^2.  Block b takes kGs2Threads m
// consecutive entries.
//
// With m = 1 and k < 128 (lz_gs2_wide_kernel) a block has four threads per
// entry, which take the vectors j = quarter (mod 4) and keep their KR values
// in registers for the update and the dot products, so that the basis is read
// once.  The kernel is a chain of dependent round trips on few blocks (45 at
// 11520 entries): all loads go out first, the partials of out in one batch,
// and a wave's dot products are folded together (wave_fold).  With one thread
// per entry it took 10.5 us a step of the Lanczos iteration on 256 boomerangs,
// now 8.0 (k < 64) and 12.4 (k = 64 .. 127, where it had read the basis twice).
constexpr int kGs2WideThreads = 4 * kGs2Threads;
// Block 0 keeps the step's first projection for the next step's first
// kernel, which publishes the step: alpha_k = c1[k] into d_ab (Lanczos), or
// all of c1 into gc1 (GMRES).
__device__ __forceinline__ void keep_c1(int k, const double* c1, double* __restrict__ d_ab,
                                        double* __restrict__ gc1) {
    if (blockIdx.x != 0) return;
    if (gc1) {
        for (int j = threadIdx.x; j <= k; j += blockDim.x) gc1[j] = c1[j];
    } else if (threadIdx.x == 0) {
        d_ab[2 * k] = c1[k];
    }
}

template <int KR>
__global__ __launch_bounds__(kGs2WideThreads) void lz_gs2_wide_kernel(
    const double* __restrict__ w, double* __restrict__ yo, int64_t n3, const double* __restrict__ V, int k,
    const double* __restrict__ part1, int ngroups, double* __restrict__ part2, double* __restrict__ d_ab,
    double* __restrict__ gc1) {
    constexpr int kWaves = kGs2Threads / 64;  // waves of one quarter
    __shared__ double c1[4 * KR];
    __shared__ double upd[4][kGs2Threads];
    __shared__ double red[kWaves][4 * KR + 1];
    const int t = threadIdx.x, el = t % kGs2Threads, qr = wave_uniform(t / kGs2Threads);
    const int64_t base = (int64_t)blockIdx.x * kGs2Threads + el;
    const bool has = base < n3;
    const unsigned bc = has ? base : 0;  // an in-bounds address for idle lanes
    // the partials of out first: the chain starts there
    RowSums<kGs2WideThreads, 8> rows;  // (16 spill)
    rows.load(part1, k + 1, ngroups);
    const double wv = w[bc];
    double a[KR];
#pragma unroll
    for (int i0 = 0; i0 < KR; i0 += 4) {
        if (4 * i0 > k) break;  // uniform
#pragma unroll
        for (int i = i0; i < i0 + 4; ++i) {
            const int j = qr + 4 * i;
            a[i] = at32(V + (j <= k ? j : 0) * n3, bc);
        }
    }
    rows.finish(part1, k + 1, ngroups, c1);
    keep_c1(k, c1, d_ab, gc1);
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < KR; ++i)
        if (qr + 4 * i <= k) s = fma(c1[qr + 4 * i], a[i], s);
    upd[qr][el] = s;
    __syncthreads();
    const double v = has ? wv - ((upd[0][el] + upd[1][el]) + (upd[2][el] + upd[3][el])) : 0.0;
    if (has && qr == 0) yo[base] = v;
    // the wave's share of the dot products of its quarter's vectors, 16 at a
    // time, and of |y'|^2
    const int wave = wave_uniform(el >> 6), lane = t & 63;
#pragma unroll
    for (int i0 = 0; i0 < KR; i0 += 16) {
        if (4 * i0 > k) break;
        double p[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) p[i] = qr + 4 * (i0 + i) <= k ? a[i0 + i] * v : 0.0;
        wave_fold<16, 32>(p);
        const int j = qr + 4 * (i0 + wave_value<16>(lane));
        if (j <= k) red[wave][j] = p[0];  // lanes with one vector write the same sum
    }
    if (qr == 0) {
        const double p = lane_group_sum<64>(v * v);
        if (lane == 0) red[wave][k + 1] = p;
    }
    __syncthreads();
    if (t < k + 2) {
        double p = red[0][t];
#pragma unroll
        for (int u = 1; u < kWaves; ++u) p += red[u][t];
        part2[(int64_t)t * gridDim.x + blockIdx.x] = p;
    }
}

// The general case: several entries per thread or many basis vectors.
__global__ __launch_bounds__(kGs2Threads) void lz_gs2_kernel(const double* __restrict__ w, double* __restrict__ yo,
                                                             int64_t n3, int m, const double* __restrict__ V, int k,
                                                             const double* __restrict__ part1, int ngroups,
                                                             double* __restrict__ part2, double* __restrict__ d_ab,
                                                             double* __restrict__ gc1) {
    constexpr int kBatch = 32;  // results per pass through the tile
    __shared__ double c1[kLanczosFusedMaxIter + 1];
    __shared__ double tile[kBatch][kGs2Threads + 1];
    const int t = threadIdx.x;
    const int nblk = gridDim.x;
    const int64_t base = (int64_t)blockIdx.x * kGs2Threads * m + t;
    const int nd = k + 2;  // V_0 .. V_k, then |y'|^2
    // the tile's kBatch rows are added by kLpr lanes each
    constexpr int kLpr = kGs2Threads / kBatch;
    const int jr = t / kLpr, c0 = t % kLpr;
    reduce_rows<kGs2Threads>(part1, k + 1, ngroups, c1);
    keep_c1(k, c1, d_ab, gc1);
    double x[kLanczosGs2PerThread];
#pragma unroll
    for (int r = 0; r < kLanczosGs2PerThread; ++r) {
        const int64_t e = base + (int64_t)r * kGs2Threads;
        x[r] = 0.0;
        if (r >= m || e >= n3) continue;
        double v = w[e], a[kPre];
        for (int j0 = 0; j0 <= k; j0 += kPre) {
#pragma unroll
            for (int j = 0; j < kPre; ++j) a[j] = j0 + j <= k ? V[(j0 + j) * n3 + e] : 0.0;
#pragma unroll
            for (int j = 0; j < kPre; ++j)
                if (j0 + j <= k) v -= c1[j0 + j] * a[j];
        }
        yo[e] = v;
        x[r] = v;
    }
    for (int j0 = 0; j0 < nd; j0 += kBatch) {
        const int jn = nd - j0 < kBatch ? nd - j0 : kBatch;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            double p = 0.0;
            if (u < jn) {
                if (j0 + u <= k) {
                    const double* av = V + (j0 + u) * n3;
#pragma unroll
                    for (int r = 0; r < kLanczosGs2PerThread; ++r) {
                        const int64_t e = base + (int64_t)r * kGs2Threads;
                        if (r < m && e < n3) p = fma(av[e], x[r], p);
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < kLanczosGs2PerThread; ++r) p = fma(x[r], x[r], p);
                }
            }
            tile[u][t] = p;
        }
        __syncthreads();
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < kGs2Threads / kLpr; ++i) s += tile[jr][c0 + kLpr * i];
        s = lane_group_sum<kLpr>(s);
        if (c0 == 0 && jr < jn) part2[(int64_t)(j0 + jr) * nblk + blockIdx.x] = s;
        __syncthreads();
    }
}

// The call's first kernel: the pair kernel's records of positions (and W
// in the force slots, which vin rewrites), B, and per block of 256 blobs
// the partial sum of |W_i|^2 (a fixed-order tree), from which vin of step 0
// forms beta_0 = |W|; block 0 also clears the definiteness flag that the
// factor build sets, which runs next.  The call's small tables (factor and
// gather offsets) come from pinned host memory with it, instead of a copy
// of their own.
template <typename R>
__global__ __launch_bounds__(kPackThreads) void lz_pack_kernel(const double* __restrict__ pos,
                                                               const double* __restrict__ W, int64_t N, int recw,
                                                               double inv_a, double lx, double ly, int64_t npad,
                                                               R* __restrict__ rec, double* __restrict__ B,
                                                               double* __restrict__ sqp, int* __restrict__ bad,
                                                               const int* __restrict__ htab, int* __restrict__ dtab,
                                                               int nwords) {
    __shared__ double red[kPackThreads];
    const int t = threadIdx.x;
    const int64_t i = (int64_t)blockIdx.x * kPackThreads + t;
    for (int64_t q = i; q < nwords; q += (int64_t)gridDim.x * kPackThreads) dtab[q] = htab[q];
    double w2 = 0.0;
    if (i < npad) {
        double b;
        make_record<R>(pos, W, N, 1, recw, inv_a, nullptr, lx, ly, i, rec + i * recw, &b);
        B[i] = b;
        if (i < N) w2 = W[3 * i] * W[3 * i] + W[3 * i + 1] * W[3 * i + 1] + W[3 * i + 2] * W[3 * i + 2];
    }
    red[t] = w2;
    __syncthreads();
    for (int h = kPackThreads / 2; h > 0; h >>= 1) {
        if (t < h) red[t] += red[t + h];
        __syncthreads();
    }
    if (t == 0) {
        sqp[blockIdx.x] = red[0];
        if (blockIdx.x == 0) *bad = 0;
    }
}

// The call's last kernel: out = L (V c) per unit (body, or run of blobs),
// with the coefficients c passed by value.
struct LzCoefs {
    double c[kLanczosCoefArgs];
};
__global__ __launch_bounds__(kVinThreads) void lz_fin_kernel(int diag, const int* __restrict__ units,
                                                             const int64_t* __restrict__ lofs,
                                                             const double* __restrict__ Lall, int64_t n3,
                                                             const double* __restrict__ V, int nv, LzCoefs cf,
                                                             double* __restrict__ out) {
    __shared__ double y[3 * kMaxBodyBlobs];
    const int p = blockIdx.x, t = threadIdx.x;
    const int64_t e0 = 3 * (int64_t)units[p];
    const int n = (int)(3 * (int64_t)units[p + 1] - e0);
    double s = 0.0;
    if (t < n) {
        const double* v = V + e0 + t;
        double s1 = 0.0;
        int j = 0;
        for (; j + 1 < nv; j += 2) {
            s = fma(cf.c[j], v[j * n3], s);
            s1 = fma(cf.c[j + 1], v[(j + 1) * n3], s1);
        }
        if (j < nv) s = fma(cf.c[j], v[j * n3], s);
        s += s1;
        y[t] = s;
    }
    __syncthreads();
    if (t < n) {
        double o;
        if (diag) {
            o = Lall[e0 + t] * s;
        } else {
            const double* Lr = Lall + 2 * lofs[p] + (int64_t)t * n;  // row t of L_p
            o = 0.0;
            for (int m = 0; m <= t; ++m) o = fma(Lr[m], y[m], o);
        }
        out[e0 + t] = o;
    }
}

}  // namespace

bool lanczos_fused_applies(int64_t N, int prec, int max_iter, const Domain& dom, SymPlan* sp) {
    if (max_iter > kLanczosFusedMaxIter) return false;
    // The symmetric plan of products of one right-hand side.  Where single
    // products take one launch (small FP64 ones) the steps take it as well, also
    // below the sizes of symmetric products: their vector work is fused with it
    // (rigid solves of 60 to 500 blobs 175 -> 120 us, roots 768 -> 494 us at 60
    // and 1593 -> 998 us at 500).
    Shape sh = tuned_shape(N, 1, prec);
    if (!dom.periodic() && !(sh.sym && sh.kblk <= 4) && !sh.direct) return false;
    if (sh.ipw < 1) sh.ipw = 4;
    if (!sh.sym && sh.direct) sh.sym = 2;
    *sp = sym_choose(N, prec, 1, sh, dom);
    return sp->ok;
}

int64_t lanczos_gs2_blocks(int64_t n3, int* m) {
    int mm = (int)((n3 + (int64_t)kGs2Threads * 1024 - 1) / ((int64_t)kGs2Threads * 1024));
    mm = std::max(1, std::min(mm, kLanczosGs2PerThread));
    *m = mm;
    return (n3 + (int64_t)kGs2Threads * mm - 1) / ((int64_t)kGs2Threads * mm);
}

// Units (blob offsets of the vin workgroups) and groups (unit offsets of the
// out workgroups: whole units of at most kLanczosOutEntries entries
// together, or one larger body alone) for bodies or, without bodies, for
// runs of kLanczosOutEntries / 3 blobs.
void lanczos_units(int64_t N, const int64_t* body_offsets, int n_bodies, std::vector<int>& units,
                   std::vector<int>& groups) {
    units.clear();
    groups.clear();
    if (n_bodies > 0) {
        for (int p = 0; p <= n_bodies; ++p) units.push_back((int)body_offsets[p]);
    } else {
        for (int64_t b = 0; b < N; b += kLanczosOutEntries / 3) units.push_back((int)b);
        units.push_back((int)N);
    }
    const int nu = (int)units.size() - 1;
    groups.push_back(0);
    int start = 0;
    for (int p = 0; p < nu; ++p) {
        if (p > start && 3 * (units[p + 1] - units[start]) > kLanczosOutEntries) {
            groups.push_back(p);
            start = p;
        }
    }
    groups.push_back(nu);
}

int lz_launch_vin(int prec, const BodyFactors& pc, const int* units, int nunits, int64_t n3, int k,
                  const double* src, const double* part2, int ncol2, double* V, double* d_ab, double* h_ab,
                  void* rec, int recw, const double* B, double* h_hdr, const int* bad0,
                  const int* bad1, hipStream_t st) {
    if (prec == RPYW_FP32C)
        hipLaunchKernelGGL(lz_vin_kernel<float>, dim3((unsigned)nunits), dim3(kVinThreads), 0, st, pc.diag ? 1 : 0,
                           units, pc.lofs, pc.L, n3, k, src, part2, ncol2, V, d_ab, h_ab, (float*)rec, recw,
                           B, h_hdr, bad0, bad1);
    else
        hipLaunchKernelGGL(lz_vin_kernel<double>, dim3((unsigned)nunits), dim3(kVinThreads), 0, st, pc.diag ? 1 : 0,
                           units, pc.lofs, pc.L, n3, k, src, part2, ncol2, V, d_ab, h_ab, (double*)rec, recw,
                           B, h_hdr, bad0, bad1);
    RPYW_HIP(hipGetLastError());
    return RPYW_OK;
}

int lz_launch_out(int prec, const BodyFactors& pc, const int* units, const LanczosGroup* ginfo, int ngroups,
                  const double* tpart, const void* spart, const SymPlan& sp, const double* B, double mu0, int64_t n3,
                  int k, const double* V, const double* d_ab, double* w, double* part1, const double* ypre,
                  hipStream_t st) {
    if (prec == RPYW_FP32C)
        hipLaunchKernelGGL(lz_out_kernel<float>, dim3((unsigned)ngroups), dim3(kOutThreads), 0, st, pc.diag ? 1 : 0,
                           units, ginfo, pc.L, tpart, (const float*)spart, sp.ng, sp.C, sp.Hmax, sp.nseg, sp.G, B,
                           mu0, n3, k, V, d_ab, w, part1, ngroups, ypre);
    else
        hipLaunchKernelGGL(lz_out_kernel<double>, dim3((unsigned)ngroups), dim3(kOutThreads), 0, st, pc.diag ? 1 : 0,
                           units, ginfo, pc.L, tpart, (const double*)spart, sp.ng, sp.C, sp.Hmax, sp.nseg, sp.G, B,
                           mu0, n3, k, V, d_ab, w, part1, ngroups, ypre);
    RPYW_HIP(hipGetLastError());
    return RPYW_OK;
}

int64_t lz_pack_blocks(int64_t npad) { return (npad + kPackThreads - 1) / kPackThreads; }

int lz_launch_pack(int prec, const double* pos, const double* W, int64_t N, int64_t npad, int recw, double a,
                   const Domain& dom, void* rec, double* B, double* sqp, int* bad, const int* htab, int* dtab,
                   int nwords, hipStream_t st) {
    const unsigned g = (unsigned)lz_pack_blocks(npad);
    if (prec == RPYW_FP32C)
        hipLaunchKernelGGL(lz_pack_kernel<float>, dim3(g), dim3(kPackThreads), 0, st, pos, W, N, recw, 1.0 / a,
                           dom.lx / a, dom.ly / a, npad, (float*)rec, B, sqp, bad, htab, dtab, nwords);
    else
        hipLaunchKernelGGL(lz_pack_kernel<double>, dim3(g), dim3(kPackThreads), 0, st, pos, W, N, recw, 1.0 / a,
                           dom.lx / a, dom.ly / a, npad, (double*)rec, B, sqp, bad, htab, dtab, nwords);
    RPYW_HIP(hipGetLastError());
    return RPYW_OK;
}

int lz_launch_fin(const BodyFactors& pc, const int* units, int nunits, int64_t n3, const double* V, const double* c,
                  int nv, double* out, hipStream_t st) {
    if (nv < 1 || nv > kLanczosCoefArgs) return RPYW_EINVAL;
    LzCoefs cf;
    for (int j = 0; j < kLanczosCoefArgs; ++j) cf.c[j] = j < nv ? c[j] : 0.0;
    hipLaunchKernelGGL(lz_fin_kernel, dim3((unsigned)nunits), dim3(kVinThreads), 0, st, pc.diag ? 1 : 0, units,
                       pc.lofs, pc.L, n3, V, nv, cf, out);
    RPYW_HIP(hipGetLastError());
    return RPYW_OK;
}

int lz_launch_gs2(const double* w, double* yo, int64_t n3, const double* V, int k, const double* part1, int ngroups,
                  double* part2, double* d_ab, double* gc1, hipStream_t st) {
    int m;
    const int64_t nb = lanczos_gs2_blocks(n3, &m);
    if (m == 1 && k < 64)
        hipLaunchKernelGGL(lz_gs2_wide_kernel<16>, dim3((unsigned)nb), dim3(kGs2WideThreads), 0, st, w, yo, n3, V, k,
                           part1, ngroups, part2, d_ab, gc1);
    else if (m == 1 && k < 128)
        hipLaunchKernelGGL(lz_gs2_wide_kernel<32>, dim3((unsigned)nb), dim3(kGs2WideThreads), 0, st, w, yo, n3, V, k,
                           part1, ngroups, part2, d_ab, gc1);
    else
        hipLaunchKernelGGL(lz_gs2_kernel, dim3((unsigned)nb), dim3(kGs2Threads), 0, st, w, yo, n3, m, V, k, part1,
                           ngroups, part2, d_ab, gc1);
    RPYW_HIP(hipGetLastError());
    return RPYW_OK;
}

}  // namespace rpyw
