// Deterministic FP64 reductions, field import/export and the fused BLAS-1 steps of CG.
#include "ks_device.h"
#include <algorithm>

#include "ks_blas.h"
#include "ks_cg_step.h"

namespace ks {

namespace {

constexpr int kFinish = 1024;

// Largest of n non-negative values: thread t takes t, t + 1024, ..., then a fixed tree.
__global__ __launch_bounds__(kFinish) void reduce_max_kernel(const double* __restrict__ in, int n,
                                                             double* __restrict__ out)
{
    double s = 0.0;
    for (int k = threadIdx.x; k < n; k += kFinish) s = fmax(s, in[k]);
    s = block_max<kFinish>(s);
    if (threadIdx.x == 0) *out = s;
}

template <int P>
__global__ __launch_bounds__(kBlock) void import_kernel(int vh, const double2* __restrict__ src,
                                                        void* __restrict__ dst)
{
    using R = typename St<P>::R;
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    if (h >= vh) return;
    cx<R> v[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double2 t = src[3 * (size_t)h + k];
        v[k] = {(R)t.x, (R)t.y};
    }
    Spinor<P>::store(dst, vh, h, v);
}

template <int P>
__global__ __launch_bounds__(kBlock) void export_kernel(int vh, const void* __restrict__ src,
                                                        double2* __restrict__ dst)
{
    using R = typename St<P>::R;
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    if (h >= vh) return;
    cx<R> v[3];
    Spinor<P>::load(src, vh, h, v);
#pragma unroll
    for (int k = 0; k < 3; ++k) dst[3 * (size_t)h + k] = make_double2((double)v[k].r, (double)v[k].i);
}

// out = in, converting storage precision
template <int PI, int PO>
__global__ __launch_bounds__(kBlock) void convert_kernel(int vh, const void* __restrict__ in,
                                                         void* __restrict__ out,
                                                         const int* __restrict__ gate)
{
    if (gate && *gate) return;
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    if (h >= vh) return;
    cx<typename St<PI>::R> v[3];
    Spinor<PI>::load(in, vh, h, v);
    cx<typename St<PO>::R> w[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) w[k] = {(typename St<PO>::R)v[k].r, (typename St<PO>::R)v[k].i};
    Spinor<PO>::store(out, vh, h, w);
}

// partial sums of |v|^2 (FP64 field)
__global__ __launch_bounds__(kBlock) void norm2_kernel(int vh, const double2* __restrict__ v,
                                                       double* __restrict__ partials)
{
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    double s = 0.0;
    if (h < vh) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double2 t = v[k * vh + h];
            s += t.x * t.x + t.y * t.y;
        }
    }
    s = block_sum<kBlock>(s);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// r = b - Ax (FP64 planes), partial sums of |r|^2
__global__ __launch_bounds__(kBlock) void sub_norm_kernel(int vh, const double2* __restrict__ b,
                                                          const double2* __restrict__ ax,
                                                          double2* __restrict__ r,
                                                          double* __restrict__ partials)
{
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    double s = 0.0;
    if (h < vh) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double2 u = b[k * vh + h], w = ax[k * vh + h];
            const double2 t = make_double2(u.x - w.x, u.y - w.y);
            r[k * vh + h] = t;
            s += t.x * t.x + t.y * t.y;
        }
    }
    s = block_sum<kBlock>(s);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// x (FP64 planes) += dx (FP32 field), dx = 0
__global__ __launch_bounds__(kBlock) void flush_dx_kernel(int vh, void* __restrict__ dx,
                                                          double2* __restrict__ x)
{
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    if (h >= vh) return;
    cx<float> d[3];
    Spinor<KS_F32>::load(dx, vh, h, d);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        double2 t = x[k * vh + h];
        t.x += (double)d[k].r;
        t.y += (double)d[k].i;
        x[k * vh + h] = t;
    }
    const cx<float> zero[3] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
    Spinor<KS_F32>::store(dx, vh, h, zero);
}

// p = r + beta p
template <int P>
__global__ __launch_bounds__(kBlock) void xpay_kernel(int vh, const void* __restrict__ r,
                                                      void* __restrict__ p,
                                                      const CGState* __restrict__ st)
{
    using R = typename St<P>::R;
    if (st->gate) return;
    const R beta = (R)st->beta;
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    if (h >= vh) return;
    cx<R> rv[3], pv[3];
    Spinor<P>::load(r, vh, h, rv);
    Spinor<P>::load(p, vh, h, pv);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        pv[k].r = fma(beta, pv[k].r, rv[k].r);
        pv[k].i = fma(beta, pv[k].i, rv[k].i);
    }
    Spinor<P>::store(p, vh, h, pv);
}

// ---------------------------------------------------------------- fused CG step

template <int P, int NT>
__global__ __launch_bounds__(NT) void cg_update_kernel(int vh, void* __restrict__ x,
                                                       const void* __restrict__ p,
                                                       const void* __restrict__ q,
                                                       void* __restrict__ r,
                                                       CGState* __restrict__ st,
                                                       const double* __restrict__ pap_part,
                                                       int npap, double* __restrict__ rr_part,
                                                       double* __restrict__ coef, int coef_cap)
{
    using R = typename St<P>::R;
    constexpr int kX = P == KS_F64 ? KS_F64 : KS_F32;
    using XR = typename St<kX>::R;
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    // one read of the gate per block: only this kernel's lead thread can change it (to 1,
    // on breakdown), and a block that sees that skips the step as the breakdown test would
    __shared__ int gated;
    if (threadIdx.x == 0) gated = st->gate;
    __syncthreads();
    if (gated) {
        if (lead) st->s_gate = 1;
        return;
    }
    double share = fused_load<NT>(pap_part, npap);
    const double rho = st->rho;
    const int h = blockIdx.x * NT + threadIdx.x;
    cx<R> pv[3], qv[3], rv[3];
    cx<XR> xv[3];
    if (h < vh) {
        Spinor<P>::load(p, vh, h, pv);
        Spinor<P>::load(q, vh, h, qv);
        Spinor<P>::load(r, vh, h, rv);
        Spinor<kX>::load(x, vh, h, xv);
        pin(pv);
        pin(qv);
        pin(rv);
        pin(xv);
    }
    const double pap = fused_total<NT>(share);
    const bool ok = isfinite(pap) && pap > 0.0;
    if (lead) {
        st->pAp = pap;
        st->s_rho = rho;
        st->s_maxr = st->maxr;
        st->s_iter = st->iter;
        st->s_gate = ok ? 0 : 1;
        if (ok) {
            st->alpha = rho / pap;
            if (st->iter < coef_cap) coef[2 * st->iter] = rho / pap;
        } else {
            st->status = isfinite(pap) ? KS_ERR_BREAKDOWN : KS_ERR_NONFINITE;
            st->gate = 1;
        }
    }
    if (!ok) return;
    const double alpha = rho / pap;
    double s = 0.0;
    if (h < vh) {
        const XR ax = (XR)alpha;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            xv[k].r = fma(ax, (XR)pv[k].r, xv[k].r);
            xv[k].i = fma(ax, (XR)pv[k].i, xv[k].i);
        }
        Spinor<kX>::store(x, vh, h, xv);
        const R a = (R)alpha;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            rv[k].r = fma(-a, qv[k].r, rv[k].r);
            rv[k].i = fma(-a, qv[k].i, rv[k].i);
        }
        Spinor<P>::store(r, vh, h, rv);
        Spinor<P>::round(rv);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            s += (double)rv[k].r * (double)rv[k].r + (double)rv[k].i * (double)rv[k].i;
    }
    s = block_sum<NT>(s);
    if (threadIdx.x == 0) rr_part[blockIdx.x] = s;
}

template <int P, int NT>
__global__ __launch_bounds__(NT) void cg_beta_xpay_kernel(int vh, const void* __restrict__ r,
                                                          void* __restrict__ p,
                                                          CGState* __restrict__ st,
                                                          const double* __restrict__ rr_part,
                                                          int nrr, double* __restrict__ coef,
                                                          int coef_cap)
{
    using R = typename St<P>::R;
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    const StepEnd end(st);
    if (end.stop) return;
    const double share = fused_load<NT>(rr_part, nrr);
    const int h = blockIdx.x * NT + threadIdx.x;
    cx<R> rv[3], pv[3];
    if (h < vh) {
        Spinor<P>::load(r, vh, h, rv);
        Spinor<P>::load(p, vh, h, pv);
        pin(rv);
        pin(pv);
    }
    double beta;
    if (!end.decide(st, fused_total<NT>(share), lead, coef, coef_cap, beta) || h >= vh) return;
    const R b = (R)beta;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        pv[k].r = fma(b, pv[k].r, rv[k].r);
        pv[k].i = fma(b, pv[k].i, rv[k].i);
    }
    Spinor<P>::store(p, vh, h, pv);
}

// ---------------------------------------------------------------- CG scalar steps

__device__ __forceinline__ double finish_sum(const double* in, int n)
{
    double s = 0.0;
    for (int k = threadIdx.x; k < n; k += kFinish) s += in[k];
    return block_sum<kFinish>(s);
}

// After r = b - A x in FP64: either converged, or continue with beta = |r|^2 / rho.
__global__ __launch_bounds__(kFinish) void cg_reliable_kernel(const double* __restrict__ part, int n,
                                                              CGState* __restrict__ st, int initial)
{
    const double r2 = finish_sum(part, n);
    if (threadIdx.x != 0) return;
    st->true_r2 = r2;
    st->ru_pending = 0;
    if (!isfinite(r2)) {
        st->status = KS_ERR_NONFINITE;
        st->gate = 1;
        return;
    }
    if (r2 <= st->stop2) {
        st->done = 1;
        st->gate = 1;
        return;
    }
    st->beta = initial ? 0.0 : r2 / st->rho;
    st->rho = r2;
    st->maxr = sqrt(r2);
    st->gate = (st->iter >= st->max_iter) ? 1 : 0;
}

__global__ void finish_to_kernel(const double* __restrict__ part, int n, double* __restrict__ out)
{
    const double s = finish_sum(part, n);
    if (threadIdx.x == 0) *out = s;
}

}  // namespace

void reduce_max(const double* partials, int n, double* out, hipStream_t s)
{
    reduce_max_kernel<<<1, kFinish, 0, s>>>(partials, n, out);
    KS_HIP(hipGetLastError());
}

void import_field(const Geom& g, ks_prec_t prec, const double* src, void* dst, hipStream_t s)
{
    const int nb = blocks_for(g.Vh);
    const double2* sp = reinterpret_cast<const double2*>(src);
    if (prec == KS_F64) import_kernel<KS_F64><<<nb, kBlock, 0, s>>>(g.Vh, sp, dst);
    else if (prec == KS_F32) import_kernel<KS_F32><<<nb, kBlock, 0, s>>>(g.Vh, sp, dst);
    else import_kernel<KS_F16><<<nb, kBlock, 0, s>>>(g.Vh, sp, dst);
    KS_HIP(hipGetLastError());
}

void export_field(const Geom& g, ks_prec_t prec, const void* src, double* dst, hipStream_t s)
{
    const int nb = blocks_for(g.Vh);
    double2* dp = reinterpret_cast<double2*>(dst);
    if (prec == KS_F64) export_kernel<KS_F64><<<nb, kBlock, 0, s>>>(g.Vh, src, dp);
    else if (prec == KS_F32) export_kernel<KS_F32><<<nb, kBlock, 0, s>>>(g.Vh, src, dp);
    else export_kernel<KS_F16><<<nb, kBlock, 0, s>>>(g.Vh, src, dp);
    KS_HIP(hipGetLastError());
}

void convert_field(int vh, ks_prec_t pin, const void* in, ks_prec_t pout, void* out,
                   const int* gate, hipStream_t s)
{
    const int nb = blocks_for(vh);
#define KS_CONV(A, B)                                                                   \
    if (pin == A && pout == B) {                                                        \
        convert_kernel<A, B><<<nb, kBlock, 0, s>>>(vh, in, out, gate);                  \
        KS_HIP(hipGetLastError());                                                      \
        return;                                                                         \
    }
    KS_CONV(KS_F64, KS_F64)
    KS_CONV(KS_F64, KS_F32)
    KS_CONV(KS_F64, KS_F16)
    KS_CONV(KS_F32, KS_F32)
    KS_CONV(KS_F32, KS_F64)
    KS_CONV(KS_F16, KS_F16)
    KS_CONV(KS_F16, KS_F64)
#undef KS_CONV
    KS_REQUIRE(false, KS_ERR_ARG, "unsupported conversion %d -> %d", (int)pin, (int)pout);
}

void norm2_partials(int vh, const double* v, double* partials, hipStream_t s)
{
    norm2_kernel<<<blocks_for(vh), kBlock, 0, s>>>(vh, reinterpret_cast<const double2*>(v), partials);
    KS_HIP(hipGetLastError());
}

void sub_norm_partials(int vh, const double* b, const double* ax, double* r, double* partials,
                       hipStream_t s)
{
    sub_norm_kernel<<<blocks_for(vh), kBlock, 0, s>>>(
        vh, reinterpret_cast<const double2*>(b), reinterpret_cast<const double2*>(ax),
        reinterpret_cast<double2*>(r), partials);
    KS_HIP(hipGetLastError());
}

int cg_step_threads(int vh) { return vh <= kCgSmall ? 256 : kCgFuse; }

namespace {

template <int P>
void launch_update(int vh, void* x, const void* p, const void* q, void* r, CGState* st,
                   const double* pap_part, int npap, double* rr_part, double* coef, int coef_cap,
                   hipStream_t s)
{
    const int nt = cg_step_threads(vh), nb = blocks_for(vh, nt);
    if (nt == 256)
        cg_update_kernel<P, 256><<<nb, 256, 0, s>>>(vh, x, p, q, r, st, pap_part, npap, rr_part,
                                                    coef, coef_cap);
    else
        cg_update_kernel<P, kCgFuse><<<nb, kCgFuse, 0, s>>>(vh, x, p, q, r, st, pap_part, npap,
                                                            rr_part, coef, coef_cap);
}

template <int P>
void launch_beta_xpay(int vh, const void* r, void* p, CGState* st, const double* rr_part,
                      double* coef, int coef_cap, hipStream_t s)
{
    const int nt = cg_step_threads(vh), nb = blocks_for(vh, nt);
    if (nt == 256)
        cg_beta_xpay_kernel<P, 256><<<nb, 256, 0, s>>>(vh, r, p, st, rr_part, nb, coef, coef_cap);
    else
        cg_beta_xpay_kernel<P, kCgFuse><<<nb, kCgFuse, 0, s>>>(vh, r, p, st, rr_part, nb, coef,
                                                               coef_cap);
}

}  // namespace

void cg_update(int vh, ks_prec_t prec, void* x, const void* p, const void* q, void* r,
               CGState* st, const double* pap_part, int npap, double* rr_part, double* coef,
               int coef_cap, hipStream_t s)
{
    if (prec == KS_F64)
        launch_update<KS_F64>(vh, x, p, q, r, st, pap_part, npap, rr_part, coef, coef_cap, s);
    else if (prec == KS_F32)
        launch_update<KS_F32>(vh, x, p, q, r, st, pap_part, npap, rr_part, coef, coef_cap, s);
    else
        launch_update<KS_F16>(vh, x, p, q, r, st, pap_part, npap, rr_part, coef, coef_cap, s);
    KS_HIP(hipGetLastError());
}

void cg_beta_xpay(int vh, ks_prec_t prec, const void* r, void* p, CGState* st,
                  const double* rr_part, double* coef, int coef_cap, hipStream_t s)
{
    if (prec == KS_F64) launch_beta_xpay<KS_F64>(vh, r, p, st, rr_part, coef, coef_cap, s);
    else if (prec == KS_F32) launch_beta_xpay<KS_F32>(vh, r, p, st, rr_part, coef, coef_cap, s);
    else launch_beta_xpay<KS_F16>(vh, r, p, st, rr_part, coef, coef_cap, s);
    KS_HIP(hipGetLastError());
}

void flush_dx(int vh, void* dx, double* x, hipStream_t s)
{
    flush_dx_kernel<<<blocks_for(vh), kBlock, 0, s>>>(vh, dx, reinterpret_cast<double2*>(x));
    KS_HIP(hipGetLastError());
}

void xpay(int vh, ks_prec_t prec, const void* r, void* p, const CGState* st, hipStream_t s)
{
    const int nb = blocks_for(vh);
    if (prec == KS_F64) xpay_kernel<KS_F64><<<nb, kBlock, 0, s>>>(vh, r, p, st);
    else if (prec == KS_F32) xpay_kernel<KS_F32><<<nb, kBlock, 0, s>>>(vh, r, p, st);
    else xpay_kernel<KS_F16><<<nb, kBlock, 0, s>>>(vh, r, p, st);
    KS_HIP(hipGetLastError());
}

void cg_reliable(const double* part, int n, CGState* st, int initial, hipStream_t s)
{
    cg_reliable_kernel<<<1, kFinish, 0, s>>>(part, n, st, initial);
    KS_HIP(hipGetLastError());
}

// Stores of the streaming read kernel land here (practically never: see there); external
// linkage keeps them, and so the loads they depend on.
__device__ unsigned g_read_sink;

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// dst = src in 16-byte units, one unit per thread, the load non-temporal (measured on gfx950:
// a one-shot grid beats grid-stride loops and multi-unit threads by 10-30 % here)
__global__ __launch_bounds__(256) void stream_copy_kernel(const u32x4* __restrict__ src,
                                                          u32x4* __restrict__ dst, size_t n)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = __builtin_nontemporal_load(src + i);
}

// Reads src in 16-byte units, one non-temporal load per thread, and folds each unit to one word;
// a lane stores only when its word equals a fixed constant, which keeps every load without
// adding traffic.  The achievable read bandwidth: the reference of the hopping term, whose
// bytes are ~98 % reads.
__global__ __launch_bounds__(256) void stream_read_kernel(const u32x4* __restrict__ src, size_t n)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const u32x4 v = __builtin_nontemporal_load(src + i);
    const unsigned w = v.x ^ v.y ^ v.z ^ v.w;
    if (w == 0x9e3779b9u) g_read_sink = w;
}

}  // namespace

void stream_copy(void* dst, const void* src, size_t bytes, hipStream_t s)
{
    const size_t n = bytes / 16;
    if (n == 0) return;
    const size_t blocks = (n + 255) / 256;
    KS_REQUIRE(blocks <= 0x7fffffffu, KS_ERR_ARG, "stream_copy: %zu bytes is too large", bytes);
    stream_copy_kernel<<<(unsigned)blocks, 256, 0, s>>>(static_cast<const u32x4*>(src),
                                                        static_cast<u32x4*>(dst), n);
    KS_HIP(hipGetLastError());
}

void stream_read(const void* src, size_t bytes, hipStream_t s)
{
    const size_t n = bytes / 16;
    if (n == 0) return;
    const size_t blocks = (n + 255) / 256;
    KS_REQUIRE(blocks <= 0x7fffffffu, KS_ERR_ARG, "stream_read: %zu bytes is too large", bytes);
    stream_read_kernel<<<(unsigned)blocks, 256, 0, s>>>(static_cast<const u32x4*>(src), n);
    KS_HIP(hipGetLastError());
}

void finish_to(const double* part, int n, double* out, hipStream_t s)
{
    finish_to_kernel<<<1, kFinish, 0, s>>>(part, n, out);
    KS_HIP(hipGetLastError());
}

}  // namespace ks
