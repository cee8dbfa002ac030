// Derivatives of u = M(r) f (arXiv:1709.02410, Sec. III: derivatives of the
// blob mobility produce the thermal drift that random finite differences
// estimate).
//
// Vector-Jacobian product for L = sum_k g_k . u_k.  With F~ = B f and
// G~ = B g (B = min(z/a, 1)) and Mhat the unregularised-height block,
//   dL/dr~_k = mu0 sum_j d1[G~_k^T Mhat(r~_k, r~_j) F~_j + F~_k^T Mhat(r~_k, r~_j) G~_j]
// (reciprocity turns the source-side appearance of r_k into the second
// form; the j = k term is then the total derivative of the self block), and
//   dL/dB_k = mu0 (g_k . (Mhat F~)_k + f_k . (Mhat G~)_k),  grad_f = mu0 B (Mhat G~).
// One fused pass per target evaluates the analytic pair gradient
// (pair_grad) and the two products; the epilogue applies the chain rule of
// the regularisation: d r~/dz = 1{z >= a}, dB/dz = 1{z < a}/a.
#include <algorithm>

#include "pair_math.h"
#include "records.h"
#include "rpyw_internal.h"
#include "sym_pairs.h"

namespace rpyw {

namespace {

constexpr int kQ = 9;  // grad (3), Mhat F~ (3), Mhat G~ (3)

template <typename R, int TILE>
__global__ __launch_bounds__(kBlock) void vjp_kernel(const R* __restrict__ rec, int64_t N, int splits,
                                                     int64_t chunk, double* __restrict__ part) {
    constexpr int RW = rec_w<R, 2>();
    constexpr int PW = pos_slots<R>();
    __shared__ __attribute__((aligned(16))) R tile[TILE * RW];
    const int b = blockIdx.x;
    const int split = b % splits;
    const int64_t first = (int64_t)(b / splits) * kBlock;
    const int64_t s0 = (int64_t)split * chunk;
    const int64_t s1 = s0 + chunk < N ? s0 + chunk : N;
    const int64_t i = first + threadIdx.x;
    const R* me = rec + (i < N ? i : N - 1) * RW;
    const R x = me[0], y = me[1], z = me[2];
    R xl = R(0), yl = R(0);
    if constexpr (sizeof(R) == 4) {
        xl = me[3];
        yl = me[4];
    }
    const R A[3] = {me[PW + 3], me[PW + 4], me[PW + 5]};   // G~ of the target
    const R A2[3] = {me[PW], me[PW + 1], me[PW + 2]};      // F~ of the target
    R acc[kQ], hi[kQ], lo[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) acc[q] = hi[q] = lo[q] = R(0);
    for (int64_t t0 = s0; t0 < s1; t0 += TILE) {
        const int n = (int)((s1 - t0) < TILE ? (s1 - t0) : TILE);
        __syncthreads();
        const R* g = rec + t0 * RW;
        for (int e = threadIdx.x; e < n * RW; e += kBlock) tile[e] = g[e];
        __syncthreads();
        for (int j = 0; j < n; ++j) {
            const R* s = tile + j * RW;
            R dx = x - s[0], dy = y - s[1];
            if constexpr (sizeof(R) == 4) {
                dx += xl - s[3];
                dy += yl - s[4];
            }
            const R dz = z - s[2];
            const R Bf[3] = {s[PW], s[PW + 1], s[PW + 2]};       // F~ of the source
            const R Bg[3] = {s[PW + 3], s[PW + 4], s[PW + 5]};   // G~ of the source
            PairCoef<R> c;
            const PairGrad<R> gr = pair_grad<R>(dx, dy, dz, z, s[2], A, Bf, A2, Bg, &c);
            acc[0] += gr.dx;
            acc[1] += gr.dy;
            acc[2] += fma_(s[2], gr.zz, gr.dz + gr.rz);
            pair_apply<R>(c, dx, dy, dz, Bf[0], Bf[1], Bf[2], acc[3], acc[4], acc[5]);
            pair_apply<R>(c, dx, dy, dz, Bg[0], Bg[1], Bg[2], acc[6], acc[7], acc[8]);
        }
        if constexpr (sizeof(R) == 4) {
#pragma unroll
            for (int q = 0; q < kQ; ++q) {
                two_sum_acc(hi[q], lo[q], acc[q]);
                acc[q] = R(0);
            }
        }
    }
    if (i >= N) return;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        const double v = sizeof(R) == 4 ? (double)hi[q] + (double)lo[q] : (double)acc[q];
        part[((int64_t)split * kQ + q) * N + i] = v;
    }
}

// The gradients of blob i from its nine sums (the chain rule of the
// regularisation).
__device__ __forceinline__ void vjp_finish(const double (&s)[kQ], const double* __restrict__ pos,
                                           const double* __restrict__ f, const double* __restrict__ g, int64_t i,
                                           double inv_a, double mu0, double* __restrict__ grad_pos,
                                           double* __restrict__ grad_f) {
    const double z = pos[3 * i + 2] * inv_a;
    const double B = z < 1.0 ? z : 1.0;
    if (grad_pos) {
        const double dLdB = mu0 * (g[3 * i] * s[3] + g[3 * i + 1] * s[4] + g[3 * i + 2] * s[5] + f[3 * i] * s[6] +
                                   f[3 * i + 1] * s[7] + f[3 * i + 2] * s[8]);
        grad_pos[3 * i] = mu0 * inv_a * s[0];
        grad_pos[3 * i + 1] = mu0 * inv_a * s[1];
        grad_pos[3 * i + 2] = z < 1.0 ? inv_a * dLdB : mu0 * inv_a * s[2];
    }
    if (grad_f)
        for (int c = 0; c < 3; ++c) grad_f[3 * i + c] = mu0 * B * s[6 + c];
}

// Epilogues: one wave per quantity of kEpiBlobs consecutive blobs, four lanes to
// a blob that share its chunks (128-byte reads).
constexpr int kEpiBlobs = 16;
constexpr int kEpiShares = 64 / kEpiBlobs;
// Adds the shares t of the lanes, finishes the blobs.
__device__ __forceinline__ void vjp_shares(double t, const double* __restrict__ pos, const double* __restrict__ f,
                                           const double* __restrict__ g, int64_t N, double inv_a, double mu0,
                                           double* __restrict__ grad_pos, double* __restrict__ grad_f) {
    __shared__ double sum[kQ][kEpiBlobs];
    const int x = threadIdx.x % kEpiBlobs;
#pragma unroll
    for (int m = kEpiBlobs; m < 64; m <<= 1) t += __shfl_xor(t, m, 64);
    if ((threadIdx.x & 63) < kEpiBlobs) sum[threadIdx.x >> 6][x] = t;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * kEpiBlobs + x;
    if (threadIdx.x >= kEpiBlobs || i >= N) return;
    double s[kQ];
#pragma unroll
    for (int k = 0; k < kQ; ++k) s[k] = sum[k][x];
    vjp_finish(s, pos, f, g, i, inv_a, mu0, grad_pos, grad_f);
}

// Of the plain kernel (below 512 blobs in FP32C, 4 to 7 chunks).  One thread per
// blob was a chain of nine sums on one or two workgroups: 10.2 us at 300 blobs,
// now 3 (a call 58.5 -> 50.6).
__global__ __launch_bounds__(64 * kQ) void vjp_epilogue(const double* __restrict__ part,
                                                        const double* __restrict__ pos, const double* __restrict__ f,
                                                        const double* __restrict__ g, int64_t N, int splits,
                                                        double inv_a, double mu0, double* __restrict__ grad_pos,
                                                        double* __restrict__ grad_f) {
    const int u = (threadIdx.x & 63) / kEpiBlobs, q = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * kEpiBlobs + threadIdx.x % kEpiBlobs;
    double t = 0.0;
    if (i < N)
        for (int p = u; p < splits; p += kEpiShares) t += part[((int64_t)p * kQ + q) * N + i];
    vjp_shares(t, pos, f, g, N, inv_a, mu0, grad_pos, grad_f);
}

// Symmetric VJP (sym_pairs.h).  For the pair (i, j) the scalar
//   Phi = G~_i^T Mhat(r~_i, r~_j) F~_j + F~_i^T Mhat(r~_i, r~_j) G~_j
// is also the pair's term seen from j (reciprocity), so one analytic pair
// gradient gives both blobs' contributions: the target derivatives for i and
// the source derivatives for j.  The two products are applied directly for i
// and transposed (wall coefficients exchanged) for j.
template <typename R>
struct VjpBody {
    static constexpr int KREC = 2;  // F~, G~
    static constexpr int NQ = kQ;   // grad (3), Mhat F~ (3), Mhat G~ (3)
    static constexpr int kUnroll = 4;
    static constexpr bool kDuo = false;
    template <bool SYM>
    __device__ static void pair(const SymTarget<R, 2>& t, const R* r, R (&acc)[kQ], R (&src)[kQ], const Box<R>&) {
        constexpr int PW = pos_slots<R>();
        R dx, dy, dz;
        sym_diff(t, r, dx, dy, dz);
        const R zj = r[2];
        const R Bf[3] = {r[PW], r[PW + 1], r[PW + 2]};
        const R Bg[3] = {r[PW + 3], r[PW + 4], r[PW + 5]};
        PairCoef<R> p;
        const PairGrad<R> g = pair_grad<R>(dx, dy, dz, t.z, zj, t.f[1], Bf, t.f[0], Bg, &p);
        acc[0] += g.dx;
        acc[1] += g.dy;
        acc[2] += fma_(zj, g.zz, g.dz + g.rz);
        pair_apply<R>(p, dx, dy, dz, Bf[0], Bf[1], Bf[2], acc[3], acc[4], acc[5]);
        pair_apply<R>(p, dx, dy, dz, Bg[0], Bg[1], Bg[2], acc[6], acc[7], acc[8]);
        if constexpr (SYM) {
            src[0] = -g.dx;
            src[1] = -g.dy;
            src[2] = fma_(t.z, g.zz, g.rz - g.dz);
            const R x = p.kcp;
            p.kcp = p.kcm;
            p.kcm = x;
#pragma unroll
            for (int q = 3; q < kQ; ++q) src[q] = R(0);
            pair_apply<R>(p, dx, dy, dz, t.f[0][0], t.f[0][1], t.f[0][2], src[3], src[4], src[5]);
            pair_apply<R>(p, dx, dy, dz, t.f[1][0], t.f[1][1], t.f[1][2], src[6], src[7], src[8]);
        }
    }
};

// Of the symmetric kernel: the four lanes share chunks and items.  Bound by the
// reads of the partials (0.53
// GB at 5e4 blobs in FP32C), and on small problems by their chain.  One thread
// per blob for all nine sums took 547 us at 5e4 blobs and 36 us at 1000 (FP64),
// one lane per blob and quantity 133 and 10.4; four lanes save another 5 us of a
// call at 1000 blobs (26.8 -> 21.6 us) and 3% at 8000.
template <typename R>
__global__ __launch_bounds__(64 * kQ) void sym_vjp_epilogue(const double* __restrict__ tpart,
                                                            const R* __restrict__ spart,
                                                            const double* __restrict__ pos,
                                                            const double* __restrict__ f,
                                                            const double* __restrict__ g, int64_t N, int ng, int C,
                                                            int Hmax, int nseg, int G, double inv_a, double mu0,
                                                            double* __restrict__ grad_pos,
                                                            double* __restrict__ grad_f) {
    const int u = (threadIdx.x & 63) / kEpiBlobs, q = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * kEpiBlobs + threadIdx.x % kEpiBlobs;
    const double t = i < N ? sym_gather<R>(tpart, spart, i, ng, C, Hmax, kQ, q, G, u, kEpiShares, nseg) : 0.0;
    vjp_shares(t, pos, f, g, N, inv_a, mu0, grad_pos, grad_f);
}

// div_i,a = sum_j sum_b d(M_ij)_ab / d r_j,b (source derivative; for j = i
// the total derivative of the self block).  One wave per target: lane l takes
// the sources j = l (mod 64), and the 64 lane sums are added in lane order,
// so the result does not depend on scheduling.  Meant for the small systems
// on which the divergence is checked (every pair costs nine gradient
// evaluations).
template <typename R>
__global__ __launch_bounds__(64) void divergence_kernel(const double* __restrict__ pos, int64_t N, double inv_a,
                                                        double mu0, double* __restrict__ div) {
    __shared__ double red[3][64];
    const int64_t i = blockIdx.x;
    const int l = threadIdx.x;
    const double xi = pos[3 * i] * inv_a, yi = pos[3 * i + 1] * inv_a, zri = pos[3 * i + 2] * inv_a;
    const double Bi = zri < 1.0 ? zri : 1.0, zti = zri < 1.0 ? 1.0 : zri;
    const double dBi = zri < 1.0 ? 1.0 : 0.0, dzti = zri < 1.0 ? 0.0 : 1.0;
    const R zero[3] = {R(0), R(0), R(0)};
    double acc[3] = {0.0, 0.0, 0.0};
    for (int64_t j = l; j < N; j += 64) {
        const double xj = pos[3 * j] * inv_a, yj = pos[3 * j + 1] * inv_a, zrj = pos[3 * j + 2] * inv_a;
        const double Bj = zrj < 1.0 ? zrj : 1.0, ztj = zrj < 1.0 ? 1.0 : zrj;
        const double dBj = zrj < 1.0 ? 1.0 : 0.0, dztj = zrj < 1.0 ? 0.0 : 1.0;
        const R dx = (R)(xi - xj), dy = (R)(yi - yj), dz = (R)(zti - ztj);
        for (int a = 0; a < 3; ++a) {
            const R ea[3] = {R(a == 0), R(a == 1), R(a == 2)};
            for (int b = 0; b < 3; ++b) {
                const R eb[3] = {R(b == 0), R(b == 1), R(b == 2)};
                PairCoef<R> c;
                const PairGrad<R> g = pair_grad<R>(dx, dy, dz, (R)zti, (R)ztj, ea, eb, zero, zero, &c);
                R u[3] = {R(0), R(0), R(0)};
                pair_apply<R>(c, dx, dy, dz, eb[0], eb[1], eb[2], u[0], u[1], u[2]);
                const double phi = (double)u[a];
                double d = 0.0;
                if (j != i) {
                    if (b == 0)
                        d = -(double)g.dx * Bi * Bj;
                    else if (b == 1)
                        d = -(double)g.dy * Bi * Bj;
                    else
                        d = Bi * (Bj * (double)(-g.dz + g.rz + (R)zti * g.zz) * dztj + dBj * phi);
                } else if (b == 2) {
                    d = 2.0 * Bi * dBi * phi + Bi * Bi * 2.0 * (double)(g.rz + (R)zti * g.zz) * dzti;
                }
                acc[a] += d;
            }
        }
    }
    for (int a = 0; a < 3; ++a) red[a][l] = acc[a];
    __syncthreads();
    if (l < 3) {
        double t = 0.0;
        for (int k = 0; k < 64; ++k) t += red[l][k];
        div[3 * i + l] = mu0 * inv_a * t;
    }
}

}  // namespace

namespace {

// Symmetric VJP plan: groups of G blobs as for the product (64 only up to
// kSym64MaxN), 9 quantities per blob.  FP64 splits the passes of few items as
// the product does, first over the four waves of a workgroup (ns), then over
// workgroups (nseg): 136 items of 64 steps left the GPU nearly empty at 1000
// blobs: 85 us a call before, 22 us now, with the records formed in the pair
// kernel (5000 blobs 317 -> 180 us).  Its 2 waves per SIMD (registers) fill
// the GPU with kVjpWaves; beyond that a split only adds partials.  FP32C is
// not split: it sums a pass in FP32, so another split is another rounding.
// Up to kVjpFusedItems items of groups of 64 the pair kernel forms the records
// itself, one launch less; that takes the FP32C kernel from 121 to 139 VGPRs,
// 3 waves per SIMD, which is as many as there are then.
constexpr int64_t kVjpWaves = 2048;
constexpr int64_t kVjpFusedItems = 3072;
struct VjpPlan {
    int G, ns, nseg, ng, C, Hmax, tail;
    size_t tb, sb;
    bool fused, ok;
};
VjpPlan vjp_sym_plan(int64_t N, int prec, int ipw, int G) {
    VjpPlan p{};
    p.G = G;
    if (G == 64 && N > kSym64MaxN) return p;
    p.ng = (int)((N + G - 1) / G);
    p.Hmax = p.ng / 2;
    p.tail = sym_tail(G, ipw, p.ng, p.Hmax);
    p.C = sym_chunks(ipw, p.Hmax, p.tail);
    const int64_t items = (int64_t)p.ng * (p.Hmax + 1);
    p.ns = (prec == RPYW_FP64 && G == 64 && items < kVjpWaves) ? 4 : 1;
    p.fused = G == 64 && items <= kVjpFusedItems;
    p.nseg = 1;
    while (p.ns > 1 && p.nseg < 4 && items * p.ns * p.nseg < kVjpWaves) p.nseg *= 2;
    p.tb = align_up((size_t)p.ng * p.C * p.nseg * kQ * G * sizeof(double));
    p.sb = align_up((size_t)p.ng * (p.Hmax + 1) * p.nseg * kQ * G * real_size(prec));
    p.ok = p.tb <= kSymPartialMaxBytes && p.sb <= kSymPartialMaxBytes;
    return p;
}

template <typename R>
void launch_vjp_sym(const R* rec, const PackSrc& ps, const VjpPlan& p, int ipw, double* tpart, R* spart,
                    hipStream_t st) {
    const dim3 grid((unsigned)(p.ng * p.C * p.nseg));
    if constexpr (sizeof(R) == 8)
        if (p.ns == 4) {
            hipLaunchKernelGGL((sym_kernel<R, VjpBody<R>, 1, 4, true>), grid, dim3(256), 0, st, rec, p.ng, p.C, ipw,
                               p.Hmax, p.nseg, tpart, spart, Box<R>{}, ps);
            return;
        }
    if (p.fused)
        hipLaunchKernelGGL((sym_kernel<R, VjpBody<R>, 1, 1, true>), grid, dim3(64), 0, st, rec, p.ng, p.C, ipw, p.Hmax,
                           p.nseg, tpart, spart, Box<R>{}, ps);
    else if (p.G == 64)
        hipLaunchKernelGGL((sym_kernel<R, VjpBody<R>, 1>), grid, dim3(64), 0, st, rec, p.ng, p.C, ipw, p.Hmax, p.nseg,
                           tpart, spart, Box<R>{}, PackSrc{});
    else
        hipLaunchKernelGGL((sym_kernel<R, VjpBody<R>, 4>), grid, dim3(256), 0, st, rec, p.ng, p.C, ipw, p.Hmax, p.nseg,
                           tpart, spart, Box<R>{}, PackSrc{}, p.tail);
}

// One symmetric VJP: records (unless fused), pairs, epilogue.
template <typename R>
int vjp_sym(const double* pos, const double* f, const double* g, double* grad_pos, double* grad_f, int64_t N, double a,
            double m0, const VjpPlan& p, int ipw, Arena& ar, hipStream_t st) {
    const int64_t npad = (int64_t)p.ng * p.G;
    double* tpart = (double*)ar.take(p.tb);
    R* spart = (R*)ar.take(p.sb);
    R* rec = nullptr;
    if (!p.fused) rec = (R*)ar.take((size_t)npad * rec_w<R, 2>() * sizeof(R));
    if (!tpart || !spart || (!p.fused && !rec)) return RPYW_ENOMEM;
    if (!p.fused) {
        hipLaunchKernelGGL(pack_kernel<R>, dim3((unsigned)((npad + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, pos, f,
                           N, 2, rec_w<R, 2>(), 1.0 / a, rec, (double*)nullptr, g, 0.0, 0.0, npad);
        RPYW_HIP(hipGetLastError());
    }
    hipEvent_t ev = nullptr;
    profile_begin(st, &ev);
    launch_vjp_sym<R>(rec, PackSrc{pos, f, N, 2, 1.0 / a, 0.0, 0.0, g}, p, ipw, tpart, spart, st);
    RPYW_HIP(hipGetLastError());
    profile_end(st, ev, (double)N * (double)N);
    hipLaunchKernelGGL(sym_vjp_epilogue<R>, dim3((unsigned)((N + kEpiBlobs - 1) / kEpiBlobs)), dim3(64 * kQ), 0, st,
                       tpart, spart, pos, f, g, N, p.ng, p.C, p.Hmax, p.nseg, p.G, 1.0 / a, m0, grad_pos, grad_f);
    RPYW_HIP(hipGetLastError());
    return RPYW_OK;
}

}  // namespace

size_t vjp_ws_bytes(int64_t N, int prec) {
    int splits;
    int64_t chunk;
    split_plan(N, 1, &splits, &chunk);
    size_t b = align_up((size_t)N * rec_width(prec, 2) * real_size(prec));
    b += align_up((size_t)N * sizeof(double));
    b += align_up((size_t)splits * kQ * N * sizeof(double));
    for (int G : {256, 64}) {
        VjpPlan p = vjp_sym_plan(N, prec, 1, G);
        if (!p.ok) p = vjp_sym_plan(N, prec, 2, G);  // as for the product
        if (p.ok)
            b = std::max(b, align_up((size_t)p.ng * G * rec_width(prec, 2) * real_size(prec)) + p.tb + p.sb);
    }
    return b + 8 * kAlign;
}

int vjp(const double* pos, const double* f, const double* g, double* grad_pos, double* grad_f, int64_t N, double a,
        double eta, int prec, Arena& ar, hipStream_t st) {
    const size_t mark = ar.used;
    const int rw = rec_width(prec, 2);
    const Shape sh = tuned_shape(N, 1, prec);
    const int ipw = sh.ipw < 1 ? 1 : sh.ipw;
    const double m0 = 1.0 / (6.0 * M_PI * eta * a);
    const unsigned g1 = (unsigned)((N + kBlock - 1) / kBlock);
    VjpPlan p{};
    if (sh.sym)
        p = vjp_sym_plan(N, prec, ipw, sym_group(sh.sym));
    else if (sh.direct)
        p = vjp_sym_plan(N, prec, 1, 64);
    if (sh.sym && !p.ok && p.G == 64) p = vjp_sym_plan(N, prec, ipw, 256);
    if (p.ok) {
        const int rc = prec == RPYW_FP32C ? vjp_sym<float>(pos, f, g, grad_pos, grad_f, N, a, m0, p, ipw, ar, st)
                                          : vjp_sym<double>(pos, f, g, grad_pos, grad_f, N, a, m0, p, ipw, ar, st);
        ar.used = mark;
        return rc;
    }
    void* rec = ar.take((size_t)N * rw * real_size(prec));
    double* B = (double*)ar.take((size_t)N * sizeof(double));
    int splits;
    int64_t chunk;
    split_plan(N, 1, &splits, &chunk);
    double* part = (double*)ar.take((size_t)splits * kQ * N * sizeof(double));
    if (!rec || !B || !part) {
        ar.used = mark;
        return RPYW_ENOMEM;
    }
    const int64_t nblocks = (int64_t)g1 * splits;
    hipEvent_t ev = nullptr;
    if (prec == RPYW_FP32C) {
        hipLaunchKernelGGL(pack_kernel<float>, dim3(g1), dim3(kBlock), 0, st, pos, f, N, 2, rw, 1.0 / a, (float*)rec, B,
                           g, 0.0, 0.0, N);
        RPYW_HIP(hipGetLastError());
        profile_begin(st, &ev);
        hipLaunchKernelGGL((vjp_kernel<float, 256>), dim3((unsigned)nblocks), dim3(kBlock), 0, st, (const float*)rec,
                           N, splits, chunk, part);
    } else {
        hipLaunchKernelGGL(pack_kernel<double>, dim3(g1), dim3(kBlock), 0, st, pos, f, N, 2, rw, 1.0 / a,
                           (double*)rec, B, g, 0.0, 0.0, N);
        RPYW_HIP(hipGetLastError());
        profile_begin(st, &ev);
        hipLaunchKernelGGL((vjp_kernel<double, 128>), dim3((unsigned)nblocks), dim3(kBlock), 0, st,
                           (const double*)rec, N, splits, chunk, part);
    }
    RPYW_HIP(hipGetLastError());
    profile_end(st, ev, (double)N * (double)N);
    hipLaunchKernelGGL(vjp_epilogue, dim3((unsigned)((N + kEpiBlobs - 1) / kEpiBlobs)), dim3(64 * kQ), 0, st, part, pos,
                       f, g, N, splits, 1.0 / a, m0, grad_pos, grad_f);
    RPYW_HIP(hipGetLastError());
    ar.used = mark;
    return RPYW_OK;
}

int divergence(const double* pos, double* div, int64_t N, double a, double eta, int prec, Arena&, hipStream_t st) {
    const unsigned g1 = (unsigned)N;  // one wave per target (N < 2^31)
    const double m0 = 1.0 / (6.0 * M_PI * eta * a);
    if (prec == RPYW_FP32C)
        hipLaunchKernelGGL(divergence_kernel<float>, dim3(g1), dim3(64), 0, st, pos, N, 1.0 / a, m0, div);
    else
        hipLaunchKernelGGL(divergence_kernel<double>, dim3(g1), dim3(64), 0, st, pos, N, 1.0 / a, m0, div);
    RPYW_HIP(hipGetLastError());
    return RPYW_OK;
}

}  // namespace rpyw
