// Batched CG: many independent lattices of uneven sizes, each with R right-hand sides, solved
// together.  One launch of each step covers every (lattice, site tile) of the batch through a
// tile table; the multi-RHS Dslash loads each link once and applies it to all R vectors of
// the site.  Every (lattice, RHS) pair keeps its own CG scalars on the device, with FP32,
// binary16 or FP64 inner iterations, FP64 solution accumulation (through FP32 increments added
// in at each reliable update in reduced precision) and per-pair FP64 reliable updates
// decided on the device, so a fixed sequence of kernels makes up one step and a run of steps
// is captured once into a HIP graph and replayed until every pair has converged.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "ks_batch.h"
#include "ks_device.h"

namespace ks {

namespace {

constexpr int kFin = 256;

// ---------------------------------------------------------------- multi-RHS vectors
// Lattice l's part of a vector arena starts at site offset vec_off_l (the sum of the Vh of the
// lattices before it) and is cut into planes of Vh_l sites with 16 bytes each (8 with one FP32
// right-hand side), so that a wave's access to a plane is one run of memory:
//   FP64: [3 colours][R] complex; FP32: [3][R / 2] pairs of complex (the right-hand sides r, r + 1);
//   binary16: [R] records {FP32 scale n, 3 x half2}, value = n * half (n = the largest real of the
//   record, as a single-RHS binary16 field stores a site).
// (With the R entries of a site adjacent instead, a lane's loads of a site lie 16 R bytes apart
// from its neighbour's and touch R times the cache lines per instruction.)
template <int P, int R>
struct MVec {
    using T = typename St<P>::R;
    static constexpr int kPer = P == KS_F64 || R == 1 ? 1 : 2;        // complex per plane entry
    static constexpr int kPlanes = 3 * R / kPer;
    using E = std::conditional_t<P == KS_F64, double2, std::conditional_t<R == 1, float2, float4>>;
    template <class B>
    __device__ static __forceinline__ auto at(B* base, size_t vec_off, int h)
    {
        using Q = std::conditional_t<std::is_const_v<B>, const E, E>;
        return reinterpret_cast<Q*>(base) + vec_off * kPlanes + h;
    }
    __device__ static __forceinline__ void load(const char* base, size_t vec_off, int vh, int h,
                                                cx<T> v[3][R])
    {
        const E* p = at(base, vec_off, h);
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int r = 0; r < R; r += kPer) {
                const E t = p[(size_t)(k * (R / kPer) + r / kPer) * vh];
                v[k][r] = {t.x, t.y};
                if constexpr (kPer == 2) v[k][r + 1] = {t.z, t.w};
            }
    }
    // v as it reads back after a store (no rounding at FP32 and FP64)
    __device__ static __forceinline__ void round(cx<T>[3][R]) {}
    __device__ static __forceinline__ void store(char* base, size_t vec_off, int vh, int h,
                                                 const cx<T> v[3][R])
    {
        E* p = at(base, vec_off, h);
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int r = 0; r < R; r += kPer) {
                E t;
                t.x = v[k][r].r;
                t.y = v[k][r].i;
                if constexpr (kPer == 2) {
                    t.z = v[k][r + 1].r;
                    t.w = v[k][r + 1].i;
                }
                p[(size_t)(k * (R / kPer) + r / kPer) * vh] = t;
            }
    }
};

template <int R>
struct MVec<KS_F16, R> {
    using T = float;
    __device__ static __forceinline__ void load(const char* base, size_t vec_off, int vh, int h,
                                                cx<T> v[3][R])
    {
        const uint4* p = reinterpret_cast<const uint4*>(base) + vec_off * R + h;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint4 q = p[(size_t)r * vh];
            const float n = __uint_as_float(q.x);
            const float2 a = unpack_half2(q.y), b = unpack_half2(q.z), c = unpack_half2(q.w);
            v[0][r] = {n * a.x, n * a.y};
            v[1][r] = {n * b.x, n * b.y};
            v[2][r] = {n * c.x, n * c.y};
        }
    }
    __device__ static __forceinline__ void store(char* base, size_t vec_off, int vh, int h,
                                                 const cx<T> v[3][R])
    {
        uint4* p = reinterpret_cast<uint4*>(base) + vec_off * R + h;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float n = 0.f;
#pragma unroll
            for (int k = 0; k < 3; ++k) n = fmaxf(n, fmaxf(fabsf(v[k][r].r), fabsf(v[k][r].i)));
            uint4 q;
            q.x = __float_as_uint(n);
            if (n > 0.f) {
                q.y = pack_half2(v[0][r].r / n, v[0][r].i / n);
                q.z = pack_half2(v[1][r].r / n, v[1][r].i / n);
                q.w = pack_half2(v[2][r].r / n, v[2][r].i / n);
            } else {
                q.y = q.z = q.w = 0u;
            }
            p[(size_t)r * vh] = q;
        }
    }
    // v replaced by the values its records decode to
    __device__ static __forceinline__ void round(cx<T> v[3][R])
    {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            cx<T> s[3] = {v[0][r], v[1][r], v[2][r]};
            Spinor<KS_F16>::round(s);
#pragma unroll
            for (int k = 0; k < 3; ++k) v[k][r] = s[k];
        }
    }
};

// The step's mode for a lattice, from the live pair fields (committed by the last kernel of
// the previous step): 2 when a pair still iterating has a reliable update due, 1 while a pair
// still iterates, 0 when every pair is done.  R <= 4: the flags of all pairs are loaded
// together, not one after another.
__device__ __forceinline__ int lattice_mode(const BatchPair* pairs, int p0, int R)
{
    int busy = 0, ru = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (r < R) {
            const BatchPair& q = pairs[p0 + r];
            busy |= !q.done;
            ru |= (!q.done && q.ru_now);
        }
    }
    return ru ? 2 : (busy ? 1 : 0);
}

// Binary16 hops of hop_site: the products of two halves are added up in FP32 by mixed-precision
// FMAs straight from the stored words (no conversion instruction, and 25 registers a hop instead
// of 42 while its loads are in flight), the record's FP32 scale times the store's enters once per
// colour.  Two hops in flight per wave at three waves per SIMD: one hop 127 us a launch, two 122,
// four 125 (32^3x48, R = 4; converted at once and scaled entry by entry: 125).
template <int R>
__device__ __forceinline__ void hop_site_f16(const LatDesc& L, int h, const int nb[16],
                                             const void* fat, const void* naik, const char* in,
                                             cx<float> res[3][R])
{
    typedef _Float16 half2v __attribute__((ext_vector_type(2)));
    const int vh = L.g.Vh, lp = L.g.lp;
    constexpr int kHops = 2;
    const uvec4* rec = reinterpret_cast<const uvec4*>(in) + L.vec_off * R;
#pragma unroll 1
    for (int s0 = 0; s0 < 16; s0 += kHops) {
        unsigned m[kHops][9];
        uvec4 v[kHops][R];
#pragma unroll
        for (int u = 0; u < kHops; ++u) {
            load_link_words(s0 < 8 ? fat : naik, (s0 + u) & 7, lp, h, m[u]);
#pragma unroll
            for (int r = 0; r < R; ++r) v[u][r] = rec[(size_t)r * vh + nb[s0 + u]];
        }
        // every load of the hops is issued before the first of their values is used
#pragma unroll
        for (int u = 0; u < kHops; ++u) {
#pragma unroll
            for (int e = 0; e < 9; ++e) asm volatile("" : "+v"(m[u][e]));
#pragma unroll
            for (int r = 0; r < R; ++r) asm volatile("" : "+v"(v[u][r]));
        }
        const float sc = s0 < 8 ? L.fat_scale : L.naik_scale;
#pragma unroll
        for (int u = 0; u < kHops; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const unsigned w[3] = {v[u][r].y, v[u][r].z, v[u][r].w};
                const float n = sc * __uint_as_float(v[u][r].x);
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    cx<float> t = {0.f, 0.f};
#pragma unroll
                    for (int b = 0; b < 3; ++b) {
                        const half2v x = __builtin_bit_cast(half2v, m[u][a * 3 + b]);
                        const half2v y = __builtin_bit_cast(half2v, w[b]);
                        cfma(t, {(float)x.x, (float)x.y}, {(float)y.x, (float)y.y});
                    }
                    res[a][r].r = fmaf(n, t.r, res[a][r].r);
                    res[a][r].i = fmaf(n, t.i, res[a][r].i);
                }
            }
    }
}

// Place of the partial sums of the tile that starts at site h0: a lattice's tiles in the order of
// their sites, whatever place the tile has in the table.  The tables' order depends on how many
// tiles the lattices before it have; the sums of a lattice, and so its solution, do not.
template <int NT>
__device__ __forceinline__ size_t part_slot(const LatDesc& L, int h0)
{
    return (size_t)(L.tile_begin + h0 / NT);
}

// res_r = (D in_r)(h) for the R right-hand sides of site h, links and vectors of precision PP.
// Hops per pass of the 16: FP32 keeps four link and neighbour loads in flight
// (measured best; a full unroll is slower); FP64 at four hops would spill.
template <int PP, int R>
__device__ __forceinline__ void hop_site(const LatDesc& L, int par, int h, const void* fat,
                                         const void* naik, const char* in,
                                         cx<typename St<PP>::R> res[3][R])
{
    using T = typename St<PP>::R;
    using V = MVec<PP, R>;
    const Geom& g = L.g;
    const int vh = g.Vh;
    int c[4];
    cb_coords(g, h, par, c);
    const int i = site_index(g, c);
    int nb[16];
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        nb[mu] = hop_cb(g, i, c, mu, +1);
        nb[4 + mu] = hop_cb(g, i, c, mu, -1);
        nb[8 + mu] = hop_cb(g, i, c, mu, +3);
        nb[12 + mu] = hop_cb(g, i, c, mu, -3);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int r = 0; r < R; ++r) res[k][r] = {0, 0};
    if constexpr (PP == KS_F16) {
        hop_site_f16<R>(L, h, nb, fat, naik, in, res);
        return;
    }
    constexpr int kHopUnroll = PP == KS_F64 ? 1 : 4;
#pragma unroll kHopUnroll
    for (int s = 0; s < 16; ++s) {
        cx<T> m[9];
        if (s < 8) load_link<PP, 9>(fat, s, g.lp, h, m);
        else load_link<PP, 9>(naik, s - 8, g.lp, h, m);
        cx<T> v[3][R];
        V::load(in, L.vec_off, vh, nb[s], v);
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
                for (int r = 0; r < R; ++r) cfma(res[a][r], m[a * 3 + b], v[b][r]);
    }
}

// The two hopping terms of a step over every (lattice, site tile): XPAY = false gives the odd
// image, XPAY = true the even output.  Per lattice, in the step's mode:
//   1 (CG step, inner precision): t = D_oe p; then q = sigma p - D_eo t with per-tile partial
//     sums of Re<p, q>;
//   2 (reliable update, FP64): t64 = D_oe x; then r64 = b - (sigma x - D_eo t64) with per-tile
//     partial sums of |r64|^2.
// Each link load serves all R right-hand sides of the site.  The second term's lead block of a
// lattice (its first tile) records the step's mode for the two kernels that follow.
template <int P, int R, bool XPAY, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void batch_hop_kernel(
    const LatDesc* __restrict__ lats, const int2* __restrict__ tiles, int ntiles, int par,
    const char* __restrict__ in, char* __restrict__ out, const char* __restrict__ xv,
    const char* __restrict__ in64, char* __restrict__ out64, const char* __restrict__ x64,
    const char* __restrict__ b64, BatchPair* __restrict__ pairs, double* __restrict__ partials)
{
    using T = typename St<P>::R;
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int2 tl = tiles[t];
        const LatDesc& L = lats[tl.x];
        const int mode = lattice_mode(pairs, L.pair0, R);
        if (XPAY && tl.y == 0 && threadIdx.x == 0) pairs[L.pair0].s_mode = mode;
        if (mode == 0) {
            if (XPAY && threadIdx.x < R) partials[part_slot<NT>(L, tl.y) * R + threadIdx.x] = 0.0;
            continue;
        }
        const int vh = L.g.Vh;
        const int h = tl.y + threadIdx.x;
        double dot[R];
#pragma unroll
        for (int r = 0; r < R; ++r) dot[r] = 0.0;
        if (h < vh) {
            if (mode == 1) {
                const void* fat = (P == KS_F64) ? L.fat64[par] : L.fat32[par];
                const void* naik = (P == KS_F64) ? L.naik64[par] : L.naik32[par];
                cx<T> res[3][R];
                hop_site<P, R>(L, par, h, fat, naik, in, res);
                if (XPAY) {
                    cx<T> xs[3][R];
                    MVec<P, R>::load(xv, L.vec_off, vh, h, xs);
#pragma unroll
                    for (int k = 0; k < 3; ++k)
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const T sg = (T)pairs[L.pair0 + r].sigma;
                            res[k][r].r = sg * xs[k][r].r - res[k][r].r;
                            res[k][r].i = sg * xs[k][r].i - res[k][r].i;
                            dot[r] += (double)xs[k][r].r * (double)res[k][r].r +
                                      (double)xs[k][r].i * (double)res[k][r].i;
                        }
                }
                MVec<P, R>::store(out, L.vec_off, vh, h, res);
            } else {
                cx<double> res[3][R];
                hop_site<KS_F64, R>(L, par, h, L.fat64[par], L.naik64[par], in64, res);
                if (XPAY) {
                    cx<double> xs[3][R], bs[3][R];
                    MVec<KS_F64, R>::load(x64, L.vec_off, vh, h, xs);
                    MVec<KS_F64, R>::load(b64, L.vec_off, vh, h, bs);
#pragma unroll
                    for (int k = 0; k < 3; ++k)
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const double sg = pairs[L.pair0 + r].sigma;
                            res[k][r].r = bs[k][r].r - (sg * xs[k][r].r - res[k][r].r);
                            res[k][r].i = bs[k][r].i - (sg * xs[k][r].i - res[k][r].i);
                            dot[r] += res[k][r].r * res[k][r].r + res[k][r].i * res[k][r].i;
                        }
                }
                MVec<KS_F64, R>::store(out64, L.vec_off, vh, h, res);
            }
        }
        if (XPAY) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const double s = block_sum<NT>(dot[r]);
                if (threadIdx.x == 0) partials[part_slot<NT>(L, tl.y) * R + r] = s;
                __syncthreads();
            }
        }
    }
}

// Sums over the lattice's tiles of the partials of every RHS (thread j adds slots j, j + NT,
// ... in order, then the fixed wave and block order): every block of the lattice gets the
// same totals bit for bit.
template <int NT, int R>
__device__ __forceinline__ void lattice_totals(const LatDesc& L, const double* __restrict__ part,
                                               double tot[4])
{
    __shared__ double red[NT / 64][4];
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    const int end = L.tile_end;
    constexpr int kAhead = 4;   // loads in flight: one 14.9 us a direction launch, four 13.3, eight 13.4
    for (int t0 = L.tile_begin + threadIdx.x; t0 < end; t0 += kAhead * NT) {
        double v[kAhead][R];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const size_t t = min(t0 + u * NT, end - 1);
#pragma unroll
            for (int r = 0; r < R; ++r) v[u][r] = part[t * R + r];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r) asm volatile("" : "+v"(v[u][r]));
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (t0 + u * NT < end)
#pragma unroll
                for (int r = 0; r < R; ++r) s[r] += v[u][r];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) s[r] = wave_sum(s[r]);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[threadIdx.x >> 6][r] = s[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < NT / 64; ++k) v += red[k][r];
        tot[r] = v;
    }
    __syncthreads();   // red is reused by the next tile
}

// The update of a step; a capped grid strides over the tiles (the lattice totals that every
// block needs are summed once per block and lattice, not once per tile).
//   mode 1: alpha = rho / <p, A p> per pair from the lattice's partials; x += alpha p (FP64 x,
//     or its FP32 increments with FP32 inner iterations), r -= alpha q, partials of |r|^2;
//     a pair with <p, A p> <= 0 or not finite stops with an error.
//   mode 2 (after r64 = b - A x): each pair finishes (|r64| at target; or the step cap, not
//     converged; or a non-finite value) or continues from r = r64 with beta = |r64|^2 / rho
//     (0 for the initial residual): p = r + beta p.
// Results for the next kernel go to the shadow fields (the lead block of the lattice).
template <int P, int R, int NT>
__global__ __launch_bounds__(NT) void batch_update_kernel(
    const LatDesc* __restrict__ lats, const int2* __restrict__ tiles, int ntiles,
    char* __restrict__ x, char* __restrict__ p, const char* __restrict__ q,
    char* __restrict__ r, const char* __restrict__ r64, BatchPair* __restrict__ pairs,
    const double* __restrict__ part, double* __restrict__ part2)
{
    using T = typename St<P>::R;
    using MV = MVec<P, R>;
    // x itself (FP64), or its FP32 increments in reduced precision
    using XV = MVec<P == KS_F64 ? KS_F64 : KS_F32, R>;
    int cached = -1;           // the lattice whose totals tot holds (the grid strides over the
    double tot[4];             // tiles, so a block's tiles mostly share a lattice)
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int2 tl = tiles[t];
        const LatDesc& L = lats[tl.x];
        const int mode = pairs[L.pair0].s_mode;
        if (mode == 0) continue;
        if (tl.x != cached) {
            lattice_totals<NT, R>(L, part, tot);
            cached = tl.x;
        }
        const bool lead = tl.y == 0 && threadIdx.x == 0;
        const int vh = L.g.Vh;
        const int h = tl.y + threadIdx.x;
        if (mode == 1) {
            double al[R];
            bool go[R];
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const BatchPair& pp = pairs[L.pair0 + k];
                const double pap = tot[k];
                const bool ok = isfinite(pap) && pap > 0.0;
                go[k] = !pp.done && ok;
                al[k] = go[k] ? pp.rho / pap : 0.0;
                if (lead) {
                    BatchPair& w = pairs[L.pair0 + k];
                    w.s_alpha = al[k];
                    w.s_done = pp.done || !ok;
                    w.s_status = (!pp.done && !ok) ? (isfinite(pap) ? KS_ERR_BREAKDOWN
                                                                    : KS_ERR_NONFINITE)
                                                   : pp.status;
                    w.s_iter = pp.iter;
                    w.s_rho = pp.rho;
                    w.s_maxr = pp.maxr;
                }
            }
            double nrm[R];
#pragma unroll
            for (int k = 0; k < R; ++k) nrm[k] = 0.0;
            if (h < vh) {
                // xv: x itself (FP64), or x's FP32 increments since the last reliable update
                cx<T> pv[3][R], qv[3][R], rv[3][R], xv[3][R];
                MV::load(p, L.vec_off, vh, h, pv);
                MV::load(q, L.vec_off, vh, h, qv);
                MV::load(r, L.vec_off, vh, h, rv);
                XV::load(x, L.vec_off, vh, h, xv);
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    // a finished pair keeps x and r: its direction is no longer maintained
                    if (!go[k]) continue;
                    const T af = (T)al[k];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        xv[c][k].r = fma(af, pv[c][k].r, xv[c][k].r);
                        xv[c][k].i = fma(af, pv[c][k].i, xv[c][k].i);
                        rv[c][k].r = fma(-af, qv[c][k].r, rv[c][k].r);
                        rv[c][k].i = fma(-af, qv[c][k].i, rv[c][k].i);
                    }
                }
                XV::store(x, L.vec_off, vh, h, xv);
                MV::store(r, L.vec_off, vh, h, rv);
                MV::round(rv);   // |r|^2 of r as stored
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    if (!go[k]) continue;
#pragma unroll
                    for (int c = 0; c < 3; ++c)
                        nrm[k] += (double)rv[c][k].r * rv[c][k].r + (double)rv[c][k].i * rv[c][k].i;
                }
            }
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const double s = block_sum<NT>(nrm[k]);
                if (threadIdx.x == 0) part2[part_slot<NT>(L, tl.y) * R + k] = s;
                __syncthreads();
            }
        } else {
            double be[R];
            bool cont[R];
            int fresh[R];
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const BatchPair& pp = pairs[L.pair0 + k];
                const double r2 = tot[k];
                const bool live = !pp.done;
                const bool fin = !isfinite(r2);
                const bool met = !fin && r2 <= pp.stop2;
                const bool cap = !fin && !met && pp.iter >= pp.max_iter;
                cont[k] = live && !fin && !met && !cap;
                fresh[k] = pp.first;
                be[k] = cont[k] ? (pp.first ? 0.0 : r2 / pp.rho) : 0.0;
                if (lead) {
                    BatchPair& w = pairs[L.pair0 + k];
                    w.s_done = pp.done || !cont[k];
                    w.s_finished = live && !cont[k];
                    w.s_status = !live ? pp.status : fin ? KS_ERR_NONFINITE
                                                        : cap ? KS_ERR_NOT_CONVERGED : pp.status;
                    w.s_true_r2 = live ? r2 : pp.true_r2;
                    w.s_ru = pp.ru + ((live && !pp.first) ? 1 : 0);
                    w.s_beta = be[k];
                    w.s_rho = cont[k] ? r2 : pp.rho;
                    w.s_maxr = cont[k] ? sqrt(r2) : pp.maxr;
                    w.s_iter = pp.iter;
                }
            }
            if (h < vh) {
                cx<double> a[3][R];
                cx<T> rv[3][R], pv[3][R];
                MVec<KS_F64, R>::load(r64, L.vec_off, vh, h, a);
                MV::load(r, L.vec_off, vh, h, rv);
                MV::load(p, L.vec_off, vh, h, pv);
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    if (!cont[k]) continue;
                    const T b = (T)be[k];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        rv[c][k] = {(T)a[c][k].r, (T)a[c][k].i};
                        if (fresh[k]) {
                            pv[c][k] = rv[c][k];
                        } else {
                            pv[c][k].r = fma(b, pv[c][k].r, rv[c][k].r);
                            pv[c][k].i = fma(b, pv[c][k].i, rv[c][k].i);
                        }
                    }
                }
                MV::store(r, L.vec_off, vh, h, rv);
                MV::store(p, L.vec_off, vh, h, pv);
            }
        }
    }
}

// The last kernel of a step (grid as for the update).
//   mode 1: |r|^2 of every pair from the lattice's partials; a pair whose residual met its
//     target or the step cap, or fell by delta since the last reliable update, asks for a
//     reliable update, and then every pair of the lattice still iterating takes it in the next
//     step (it costs the lattice one FP64 multi-RHS A-apply whatever the number of pairs):
//     x's FP32 increments are added into x here.  Otherwise p = r + beta p, beta = |r|^2 / rho.
//   mode 2: the reliable update's results are committed.
// The lead block commits the live fields of the lattice's pairs from the shadows.
template <int P, int R, int NT>
__global__ __launch_bounds__(NT) void batch_direction_kernel(
    const LatDesc* __restrict__ lats, const int2* __restrict__ tiles, int ntiles,
    const char* __restrict__ r, char* __restrict__ p, char* __restrict__ x64,
    char* __restrict__ dx, BatchPair* __restrict__ pairs, const double* __restrict__ part2)
{
    using T = typename St<P>::R;
    using MV = MVec<P, R>;
    int cached = -1;
    double tot[4];
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int2 tl = tiles[t];
        const LatDesc& L = lats[tl.x];
        const int mode = pairs[L.pair0].s_mode;
        if (mode == 0) continue;
        const bool lead = tl.y == 0 && threadIdx.x == 0;
        if (mode == 2) {
            if (lead) {
                const unsigned long long now = wall_clock64();
                for (int k = 0; k < R; ++k) {
                    BatchPair& w = pairs[L.pair0 + k];
                    if (w.done) continue;
                    w.done = w.s_done;
                    w.status = w.s_status;
                    w.true_r2 = w.s_true_r2;
                    w.ru = w.s_ru;
                    w.beta = w.s_beta;
                    w.rho = w.s_rho;
                    w.maxr = w.s_maxr;
                    w.ru_now = 0;
                    w.first = 0;
                    if (w.s_finished) w.t_done = now;
                }
            }
            continue;
        }
        if (tl.x != cached) {
            lattice_totals<NT, R>(L, part2, tot);
            cached = tl.x;
        }
        bool live[R], nonfin[R], due[R];
        bool any_due = false;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const BatchPair& pp = pairs[L.pair0 + k];
            const double rn = tot[k];
            live[k] = !pp.s_done;
            nonfin[k] = live[k] && !isfinite(rn);
            const bool met = rn <= pp.stop2 || pp.s_iter + 1 >= pp.max_iter;
            const bool fell = sqrt(rn) < pp.delta * pp.s_maxr;
            due[k] = live[k] && !nonfin[k] && (met || fell);
            any_due = any_due || due[k];
        }
        const int vh = L.g.Vh;
        const int h = tl.y + threadIdx.x;
        if (h < vh) {
            if (any_due) {
                if (P != KS_F64 && dx) {
                    cx<double> xv[3][R];
                    cx<float> dv[3][R], zero[3][R];
                    MVec<KS_F64, R>::load(x64, L.vec_off, vh, h, xv);
                    MVec<KS_F32, R>::load(dx, L.vec_off, vh, h, dv);
#pragma unroll
                    for (int c = 0; c < 3; ++c)
#pragma unroll
                        for (int k = 0; k < R; ++k) {
                            xv[c][k].r += (double)dv[c][k].r;
                            xv[c][k].i += (double)dv[c][k].i;
                            zero[c][k] = {0.f, 0.f};
                        }
                    MVec<KS_F64, R>::store(x64, L.vec_off, vh, h, xv);
                    MVec<KS_F32, R>::store(dx, L.vec_off, vh, h, zero);
                }
            } else {
                cx<T> rv[3][R], pv[3][R];
                MV::load(r, L.vec_off, vh, h, rv);
                MV::load(p, L.vec_off, vh, h, pv);
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    if (!live[k] || nonfin[k]) continue;
                    const T b = (T)(tot[k] / pairs[L.pair0 + k].s_rho);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        pv[c][k].r = fma(b, pv[c][k].r, rv[c][k].r);
                        pv[c][k].i = fma(b, pv[c][k].i, rv[c][k].i);
                    }
                }
                MV::store(p, L.vec_off, vh, h, pv);
            }
        }
        if (lead) {
            const unsigned long long now = wall_clock64();
            for (int k = 0; k < R; ++k) {
                BatchPair& w = pairs[L.pair0 + k];
                if (w.done) continue;
                w.alpha = w.s_alpha;
                if (w.s_done) {   // <p, A p> broke down in the update
                    w.done = 1;
                    w.status = w.s_status;
                    w.t_done = now;
                    continue;
                }
                w.iter = w.s_iter + 1;
                const double rn = tot[k];
                if (nonfin[k]) {
                    w.done = 1;
                    w.status = KS_ERR_NONFINITE;
                    w.t_done = now;
                } else if (any_due) {
                    w.ru_now = due[k] ? 2 : 1;
                } else {
                    w.beta = rn / w.s_rho;
                    w.rho = rn;
                    w.maxr = fmax(w.s_maxr, sqrt(rn));
                }
            }
        }
    }
}

// FP32 inner: x += dx, dx = 0 on every lattice (the remaining increments at the end)
template <int R, int NT>
__global__ __launch_bounds__(NT) void batch_flush_kernel(const LatDesc* __restrict__ lats,
                                                        const int2* __restrict__ tiles, int ntiles,
                                                        char* __restrict__ x, char* __restrict__ dx)
{
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int2 tl = tiles[t];
        const LatDesc& L = lats[tl.x];
        const int vh = L.g.Vh;
        const int h = tl.y + threadIdx.x;
        if (h >= vh) continue;
        cx<double> xv[3][R];
        cx<float> dv[3][R], zero[3][R];
        MVec<KS_F64, R>::load(x, L.vec_off, vh, h, xv);
        MVec<KS_F32, R>::load(dx, L.vec_off, vh, h, dv);
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int k = 0; k < R; ++k) {
                xv[c][k].r += (double)dv[c][k].r;
                xv[c][k].i += (double)dv[c][k].i;
                zero[c][k] = {0.f, 0.f};
            }
        MVec<KS_F64, R>::store(x, L.vec_off, vh, h, xv);
        MVec<KS_F32, R>::store(dx, L.vec_off, vh, h, zero);
    }
}

// One block per pair: its lattice's tile partials in slot order.
__device__ __forceinline__ double pair_sum(const LatDesc& L, const double* part, int R, int r)
{
    double s = 0.0;
    for (int t = L.tile_begin + threadIdx.x; t < L.tile_end; t += kFin) s += part[(size_t)t * R + r];
    return block_sum<kFin>(s);
}

__global__ void batch_census_kernel(const BatchPair* __restrict__ pairs, int n, int* __restrict__ out)
{
    __shared__ int cnt;
    if (threadIdx.x == 0) cnt = 0;
    __syncthreads();
    int c = 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) c += pairs[i].done ? 1 : 0;
    atomicAdd(&cnt, c);
    __syncthreads();
    if (threadIdx.x == 0) *out = cnt;
}

__global__ void batch_clock_kernel(unsigned long long* out) { *out = wall_clock64(); }

// Per tile: partial sums of |b_r|^2 over its sites, for every RHS r (FP64 arena).
template <int R, int NT>
__global__ __launch_bounds__(NT) void batch_b2_kernel(const LatDesc* __restrict__ lats,
                                                     const int2* __restrict__ tiles,
                                                     const char* __restrict__ b64,
                                                     double* __restrict__ partials)
{
    const int t = blockIdx.x;
    const int2 tl = tiles[t];
    const LatDesc& L = lats[tl.x];
    const int vh = L.g.Vh;
    const int h = tl.y + threadIdx.x;
    double nrm[R];
#pragma unroll
    for (int k = 0; k < R; ++k) nrm[k] = 0.0;
    if (h < vh) {
        cx<double> v[3][R];
        MVec<KS_F64, R>::load(b64, L.vec_off, vh, h, v);
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int k = 0; k < R; ++k) nrm[k] += v[c][k].r * v[c][k].r + v[c][k].i * v[c][k].i;
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const double s = block_sum<NT>(nrm[k]);
        if (threadIdx.x == 0) partials[part_slot<NT>(L, tl.y) * R + k] = s;
        __syncthreads();
    }
}

// Per pair: |b|^2 (the tile partials in slot order) and the initial scalars (one block per pair).
__global__ __launch_bounds__(kFin) void batch_init_pairs_kernel(const LatDesc* __restrict__ lats,
                                                                int R, BatchPair* __restrict__ pairs,
                                                                const double* __restrict__ part,
                                                                const double* __restrict__ param,
                                                                int npairs, double delta,
                                                                int max_iter,
                                                                double* __restrict__ b2_out)
{
    const int pi = blockIdx.x;
    const LatDesc& L = lats[pi / R];
    const double s = pair_sum(L, part, R, pi % R);
    if (threadIdx.x != 0) return;
    BatchPair q{};
    q.sigma = param[pi];
    const double tol = param[npairs + pi];
    q.stop2 = tol * tol * s;
    q.delta = delta;
    q.max_iter = max_iter;
    q.ru_now = (s > 0.0) ? 1 : 0;   // the initial residual is the first step's FP64 update
    q.first = 1;
    q.done = (s > 0.0) ? 0 : 1;
    pairs[pi] = q;
    b2_out[pi] = s;
}

// Caller vectors (complex128 [Vh][3], one device pointer per pair) <-> arena slots.
template <int R>
__global__ void batch_io_kernel(const LatDesc* __restrict__ lats, char* __restrict__ arena,
                                void* const* __restrict__ ptrs, int to_arena)
{
    const int pi = blockIdx.y;
    const LatDesc& L = lats[pi / R];
    const int r = pi % R;
    const int vh = L.g.Vh;
    double2* u = static_cast<double2*>(ptrs[pi]);
    for (int h = blockIdx.x * blockDim.x + threadIdx.x; h < vh; h += gridDim.x * blockDim.x) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            double2* a = MVec<KS_F64, R>::at(arena, L.vec_off, h) + (size_t)(k * R + r) * vh;
            if (to_arena) *a = u[(size_t)h * 3 + k];
            else u[(size_t)h * 3 + k] = *a;
        }
    }
}

}  // namespace

// ---------------------------------------------------------------- launchers

// Most threads of the update and direction kernels' grids, which stride over the tiles (eight waves
// per SIMD, some three times what is resident; set by measurement).  Every block sums its lattices' partials once per lattice it meets, so
// fewer blocks than tiles pay on one large lattice (3072 tiles of 256, binary16, R = 4: 62 + 36 us
// against 66 + 39 with a block per tile), while a batch whose tiles all fit takes a block per tile
// (3212 tiles of 64, FP32, R = 4: 23.1 + 14.3 us, 24.5 + 16.7 with 2048 blocks).
constexpr int kUpdateThreads = 2048 * 256;

template <int R, int NT>
struct BatchLaunch {
    // a hopping term of the step: odd image (xpay = false) or even output (xpay = true)
    static void hop(BatchCtx& c, bool xpay, hipStream_t s)
    {
        const int nt = c.ntiles[c.tile_idx];
        const int2* tl = c.tiles[c.tile_idx];
        const int grid = c.grid(nt);
#define KS_BH(P, X)                                                                            \
    batch_hop_kernel<P, R, X, NT><<<grid, NT, 0, s>>>(                                          \
        c.lats_dev, tl, nt, X ? 0 : 1, X ? c.ts : c.ps, X ? c.qs : c.ts, c.ps,                  \
        X ? c.t64 : c.x64, X ? c.r64 : c.t64, c.x64, c.b64, c.pairs, c.partials)
        if (c.prec == KS_F64) {
            if (xpay) KS_BH(KS_F64, true);
            else KS_BH(KS_F64, false);
        } else if (c.prec == KS_F16) {
            if (xpay) KS_BH(KS_F16, true);
            else KS_BH(KS_F16, false);
        } else {
            if (xpay) KS_BH(KS_F32, true);
            else KS_BH(KS_F32, false);
        }
#undef KS_BH
        KS_HIP(hipGetLastError());
    }
    // one step: two hopping terms, the update, the direction update (four launches)
    static void step(BatchCtx& c, hipStream_t s)
    {
        const int nt = c.ntiles[c.tile_idx];
        const int2* tl = c.tiles[c.tile_idx];
        hop(c, false, s);
        hop(c, true, s);
        // the update kernels stride over the tiles with a capped grid: every block sums its
        // lattices' partials, once per lattice it meets
        const int ug = std::min(nt, kUpdateThreads / NT);
        if (c.prec == KS_F64) {
            batch_update_kernel<KS_F64, R, NT><<<ug, NT, 0, s>>>(c.lats_dev, tl, nt, c.x64, c.ps,
                                                                 c.qs, c.rs, c.r64, c.pairs,
                                                                 c.partials, c.partials2);
            batch_direction_kernel<KS_F64, R, NT><<<ug, NT, 0, s>>>(c.lats_dev, tl, nt, c.rs,
                                                                    c.ps, c.x64, nullptr, c.pairs,
                                                                    c.partials2);
        } else if (c.prec == KS_F16) {
            batch_update_kernel<KS_F16, R, NT><<<ug, NT, 0, s>>>(c.lats_dev, tl, nt, c.dx32, c.ps,
                                                                 c.qs, c.rs, c.r64, c.pairs,
                                                                 c.partials, c.partials2);
            batch_direction_kernel<KS_F16, R, NT><<<ug, NT, 0, s>>>(c.lats_dev, tl, nt, c.rs,
                                                                    c.ps, c.x64, c.dx32, c.pairs,
                                                                    c.partials2);
        } else {
            batch_update_kernel<KS_F32, R, NT><<<ug, NT, 0, s>>>(c.lats_dev, tl, nt, c.dx32, c.ps,
                                                                 c.qs, c.rs, c.r64, c.pairs,
                                                                 c.partials, c.partials2);
            batch_direction_kernel<KS_F32, R, NT><<<ug, NT, 0, s>>>(c.lats_dev, tl, nt, c.rs,
                                                                    c.ps, c.x64, c.dx32, c.pairs,
                                                                    c.partials2);
        }
        KS_HIP(hipGetLastError());
    }
    static void flush(BatchCtx& c, hipStream_t s)
    {
        const int nt = c.ntiles[c.tile_idx];
        batch_flush_kernel<R, NT><<<nt, NT, 0, s>>>(c.lats_dev, c.tiles[c.tile_idx], nt, c.x64,
                                                    c.dx32);
        KS_HIP(hipGetLastError());
    }
    static void b2(BatchCtx& c, hipStream_t s)
    {
        const int nt = c.ntiles[c.tile_idx];
        batch_b2_kernel<R, NT><<<nt, NT, 0, s>>>(c.lats_dev, c.tiles[c.tile_idx], c.b64, c.partials);
        KS_HIP(hipGetLastError());
    }
};

static const int kTileSizes[3] = {64, 128, 256};

template <int R>
static void dispatch(BatchCtx& c, int what, hipStream_t s)
{
    const int nt = kTileSizes[c.tile_idx];
#define KS_DISP(NTV)                                                                    \
    if (nt == NTV) {                                                                    \
        if (what == 0) BatchLaunch<R, NTV>::step(c, s);                                 \
        else if (what == 3) BatchLaunch<R, NTV>::b2(c, s);                              \
        else if (what == 4) BatchLaunch<R, NTV>::flush(c, s);                           \
        else BatchLaunch<R, NTV>::hop(c, false, s);                                     \
        return;                                                                         \
    }
    KS_DISP(64)
    KS_DISP(128)
    KS_DISP(256)
#undef KS_DISP
}

static void run(BatchCtx& c, int what, hipStream_t s)
{
    switch (c.nrhs) {
    case 1: dispatch<1>(c, what, s); break;
    case 2: dispatch<2>(c, what, s); break;
    case 4: dispatch<4>(c, what, s); break;
    default: KS_REQUIRE(false, KS_ERR_ARG, "batch: nrhs must be 1, 2 or 4");
    }
}

int BatchCtx::grid(int ntiles_now) const
{
    return persistent > 0 ? std::min(ntiles_now, persistent) : ntiles_now;
}

void batch_free(BatchCtx* c)
{
    if (!c) return;
    if (c->graph_exec) (void)hipGraphExecDestroy(c->graph_exec);
    if (c->owns_gauges)
        for (ks_gauge_t g : c->gauges) {
            gauge_release(g);
            delete g;
        }
    device_free(c->lats_dev);
    for (int k = 0; k < 3; ++k) device_free(c->tiles[k]);
    device_free(c->partials);
    device_free(c->partials2);
    device_free(c->pairs);
    device_free(c->clock);
    device_free(c->census);
    device_free(c->b2);
    device_free(c->pair_param);
    device_free(c->io_ptrs);
    for (char* v : {c->ps, c->qs, c->ts, c->rs, c->x64, c->b64, c->r64, c->t64, c->ax64, c->dx32})
        device_free(v);
    if (c->pairs_host) (void)hipHostFree(c->pairs_host);
    if (c->census_host) (void)hipHostFree(c->census_host);
    if (c->order) (void)hipEventDestroy(c->order);
    if (c->stream) (void)hipStreamDestroy(c->stream);
    delete c;
}

// Lattice descriptors, tile tables, pair state and vector arenas for the gauges of c.
static void batch_setup(BatchCtx* c, hipStream_t s)
{
    const int nlat = (int)c->gauges.size();
    const int nrhs = c->nrhs;
    const ks_prec_t inner = c->prec;
    size_t vec_off = 0;
    std::vector<LatDesc> lats(nlat);
    for (int l = 0; l < nlat; ++l) {
        ks_gauge_t g = c->gauges[l];
        if (inner != KS_F64) gauge_prepare(g, inner, KS_RECON_18, s);
        LatDesc& L = lats[l];
        L.g = g->geom;
        for (int par = 0; par < 2; ++par) {
            L.fat64[par] = g->store[KS_F64][0].fat[par];
            L.naik64[par] = g->store[KS_F64][0].naik[par];
            L.fat32[par] = g->store[inner][0].fat[par];
            L.naik32[par] = g->store[inner][0].naik[par];
        }
        L.fat_scale = g->store[inner][0].fat_scale;
        L.naik_scale = g->store[inner][0].naik_scale;
        L.vec_off = vec_off;
        L.pair0 = l * nrhs;
        vec_off += (size_t)g->geom.Vh;
    }
    c->total_vh = vec_off;
    // tile tables for 64, 128 and 256 sites per tile.  Blocks go round robin to the eight XCDs, and
    // the vectors of R right-hand sides are most of what an L2 could hold between their reads by
    // neighbouring sites: each XCD gets an eighth of every lattice (so that it keeps work while
    // any lattice iterates), in columns of kColumn z-planes walked along t.  32^3x48, binary16,
    // R = 4: the hopping term's two launches 122 + 130 us in index order, 131 + 131 with eighths alone,
    // 121 + 127 / 120 + 126 / 119 + 126 / 119 + 126 / 126 + 127 with columns of 1 / 2 / 4 / 8 / 16
    // planes; update and direction, which meet their tiles in the same L2: 66 + 36.5 to 64 + 35.6.
    constexpr int kColumn = 4;
    size_t max_tiles = 0;
    for (int k = 0; k < 3; ++k) {
        std::vector<int2> tt;
        for (int l = 0; l < nlat; ++l) {
            if (k == 0) lats[l].tile_begin = (int)tt.size();
            const Geom& g = lats[l].g;
            std::vector<int> seq;
            for (int h0 = 0; h0 < g.Vh; h0 += kTileSizes[k]) seq.push_back(h0);
            const int plane = g.n[0] / 2 * g.n[1];
            auto walk = [&](int h0) {
                const int z = h0 / plane % g.n[2], t = h0 / plane / g.n[2];
                return std::make_pair(z / kColumn * g.n[3] + t, h0);
            };
            std::sort(seq.begin(), seq.end(), [&](int a, int b) { return walk(a) < walk(b); });
            const size_t t0 = tt.size();
            tt.resize(t0 + seq.size());
            size_t at = 0;
            for (size_t xcd = 0; xcd < 8; ++xcd)
                for (size_t t = t0; t < tt.size(); ++t)
                    if ((t & 7) == xcd) tt[t] = make_int2(l, seq[at++]);
        }
        c->ntiles[k] = (int)tt.size();
        c->tiles[k] = static_cast<int2*>(device_alloc(sizeof(int2) * tt.size()));
        KS_HIP(hipMemcpyAsync(c->tiles[k], tt.data(), sizeof(int2) * tt.size(),
                              hipMemcpyHostToDevice, s));
        max_tiles = std::max(max_tiles, tt.size());
        c->tile_tables[k] = tt;
    }
    c->lats_host = lats;
    c->lats_dev = static_cast<LatDesc*>(device_alloc(sizeof(LatDesc) * nlat));
    c->set_tiles(0, s);
    c->partials = static_cast<double*>(device_alloc(sizeof(double) * max_tiles * nrhs));
    c->partials2 = static_cast<double*>(device_alloc(sizeof(double) * max_tiles * nrhs));
    c->pairs = static_cast<BatchPair*>(device_alloc(sizeof(BatchPair) * c->npairs));
    KS_HIP(hipHostMalloc(reinterpret_cast<void**>(&c->pairs_host), sizeof(BatchPair) * c->npairs));
    c->clock = static_cast<unsigned long long*>(device_alloc(sizeof(unsigned long long)));
    c->census = static_cast<int*>(device_alloc(sizeof(int)));
    c->b2 = static_cast<double*>(device_alloc(sizeof(double) * c->npairs));
    c->pair_param = static_cast<double*>(device_alloc(sizeof(double) * 2 * c->npairs));
    c->io_ptrs = static_cast<void**>(device_alloc(sizeof(void*) * c->npairs));
    KS_HIP(hipHostMalloc(reinterpret_cast<void**>(&c->census_host), sizeof(int)));
    const size_t cs = inner == KS_F64 ? 16 : 8;
    const size_t nrec = vec_off * 3 * nrhs;
    // inner-precision arenas: complex numbers of cs bytes, or one 16-byte binary16 record per
    // site and right-hand side
    const size_t ib = inner == KS_F16 ? vec_off * nrhs * 16 : nrec * cs;
    c->inner_bytes = ib;
    c->ps = static_cast<char*>(device_alloc(ib));
    c->qs = static_cast<char*>(device_alloc(ib));
    c->ts = static_cast<char*>(device_alloc(ib));
    c->rs = static_cast<char*>(device_alloc(ib));
    c->x64 = static_cast<char*>(device_alloc(nrec * 16));
    c->b64 = static_cast<char*>(device_alloc(nrec * 16));
    c->r64 = static_cast<char*>(device_alloc(nrec * 16));
    c->t64 = static_cast<char*>(device_alloc(nrec * 16));
    c->ax64 = static_cast<char*>(device_alloc(nrec * 16));
    if (inner != KS_F64) {
        c->dx32_bytes = nrec * 8;
        c->dx32 = static_cast<char*>(device_alloc(c->dx32_bytes));
    }
    // finished pairs leave their slots of p, q, t untouched: start every arena finite
    for (char* a : {c->ps, c->qs, c->ts, c->rs})
        KS_HIP(hipMemsetAsync(a, 0, ib, s));
    for (char* a : {c->x64, c->b64, c->r64, c->t64, c->ax64})
        KS_HIP(hipMemsetAsync(a, 0, nrec * 16, s));
    KS_HIP(hipStreamSynchronize(s));
}

static BatchCtx* batch_new(int nrhs, ks_prec_t inner)
{
    KS_REQUIRE(nrhs == 1 || nrhs == 2 || nrhs == 4, KS_ERR_ARG, "batch: nrhs must be 1, 2 or 4");
    KS_REQUIRE(inner == KS_F64 || inner == KS_F32 || inner == KS_F16, KS_ERR_ARG,
               "batch: inner precision F64, F32 or F16");
    BatchCtx* c = new BatchCtx();
    c->nrhs = nrhs;
    c->prec = inner;
    try {
        KS_HIP(hipStreamCreateWithFlags(&c->stream, hipStreamNonBlocking));
        KS_HIP(hipEventCreateWithFlags(&c->order, hipEventDisableTiming));
    } catch (...) {
        batch_free(c);
        throw;
    }
    return c;
}

BatchCtx* batch_create(int nlat, const int* dims, const double* const* fat,
                       const double* const* naik, int on_device, int nrhs, ks_prec_t inner,
                       hipStream_t s)
{
    KS_REQUIRE(nlat >= 1, KS_ERR_ARG, "batch: no lattices");
    BatchCtx* c = batch_new(nrhs, inner);
    try {
        c->npairs = nlat * nrhs;
        for (int l = 0; l < nlat; ++l) {
            const int* d = dims + 4 * l;
            long v = 1;
            for (int mu = 0; mu < 4; ++mu) {
                KS_REQUIRE(d[mu] >= 4 && d[mu] % 2 == 0, KS_ERR_ARG,
                           "batch lattice %d: extent %d of direction %d must be even and >= 4", l,
                           d[mu], mu);
                v *= d[mu];
            }
            KS_REQUIRE(v <= (1L << 29), KS_ERR_ARG, "batch lattice %d: volume too large", l);
            KS_REQUIRE(fat[l] && naik[l], KS_ERR_ARG, "batch lattice %d: null links", l);
            ks_gauge_s* g = new ks_gauge_s();
            c->gauges.push_back(g);
            g->geom = make_geom(d);
            const size_t bytes = (size_t)4 * v * 9 * 16;
            const double* df = fat[l];
            const double* dn = naik[l];
            double* tf = nullptr;
            double* tn = nullptr;
            if (!on_device) {
                tf = static_cast<double*>(device_alloc(bytes));
                tn = static_cast<double*>(device_alloc(bytes));
                KS_HIP(hipMemcpyAsync(tf, fat[l], bytes, hipMemcpyHostToDevice, s));
                KS_HIP(hipMemcpyAsync(tn, naik[l], bytes, hipMemcpyHostToDevice, s));
                df = tf;
                dn = tn;
            }
            gauge_build_f64(g, df, dn, s);
            device_free(tf);
            device_free(tn);
        }
        batch_setup(c, s);
    } catch (...) {
        batch_free(c);
        throw;
    }
    return c;
}

BatchCtx* batch_create_on(ks_gauge_t g, int nrhs, ks_prec_t inner, hipStream_t s)
{
    BatchCtx* c = batch_new(nrhs, inner);
    try {
        c->owns_gauges = false;
        c->npairs = nrhs;
        c->gauges.push_back(g);
        batch_setup(c, s);
    } catch (...) {
        batch_free(c);
        throw;
    }
    return c;
}

void BatchCtx::set_tiles(int k, hipStream_t s)
{
    tile_idx = k;
    std::vector<LatDesc> l = lats_host;
    const std::vector<int2>& tt = tile_tables[k];
    for (size_t i = 0; i < l.size(); ++i) {
        l[i].tile_begin = -1;
        l[i].tile_end = -1;
    }
    for (size_t t = 0; t < tt.size(); ++t) {
        LatDesc& L = l[tt[t].x];
        if (L.tile_begin < 0) L.tile_begin = (int)t;
        L.tile_end = (int)t + 1;
    }
    lats_host = l;
    KS_HIP(hipMemcpyAsync(lats_dev, l.data(), sizeof(LatDesc) * l.size(), hipMemcpyHostToDevice, s));
    KS_HIP(hipStreamSynchronize(s));
    if (graph_exec) {
        (void)hipGraphExecDestroy(graph_exec);
        graph_exec = nullptr;
    }
}

// Caller vectors <-> arena: one launch for every pair through a device pointer table.
static void batch_io(BatchCtx& c, char* arena, const void* const* host_ptrs, int to_arena,
                     hipStream_t s)
{
    KS_HIP(hipMemcpyAsync(c.io_ptrs, host_ptrs, sizeof(void*) * c.npairs, hipMemcpyHostToDevice, s));
    int maxvh = 0;
    for (const LatDesc& L : c.lats_host) maxvh = std::max(maxvh, L.g.Vh);
    const dim3 grid(std::min(blocks_for(maxvh), 64), c.npairs);
    if (c.nrhs == 1) batch_io_kernel<1><<<grid, kBlock, 0, s>>>(c.lats_dev, arena, c.io_ptrs, to_arena);
    else if (c.nrhs == 2) batch_io_kernel<2><<<grid, kBlock, 0, s>>>(c.lats_dev, arena, c.io_ptrs, to_arena);
    else batch_io_kernel<4><<<grid, kBlock, 0, s>>>(c.lats_dev, arena, c.io_ptrs, to_arena);
    KS_HIP(hipGetLastError());
    // the pointer table is read by the kernel: keep it until the copy has been consumed
    KS_HIP(hipStreamSynchronize(s));
}

// The batch runs on its own stream (graphs cannot be captured on the legacy default stream),
// ordered after the caller's stream.
static hipStream_t enter_stream(BatchCtx& c, hipStream_t caller)
{
    KS_HIP(hipEventRecord(c.order, caller));
    KS_HIP(hipStreamWaitEvent(c.stream, c.order, 0));
    return c.stream;
}

ks_status_t batch_solve(BatchCtx& c, const double* masses, const double* const* b,
                        double* const* x, const ks_solver_params& prm, ks_batch_stats* stats,
                        hipStream_t caller)
{
    const int nlat = (int)c.lats_host.size();
    std::vector<double> sigma(c.npairs), tol(c.npairs, prm.tol);
    for (int l = 0; l < nlat; ++l) {
        KS_REQUIRE(std::isfinite(masses[l]), KS_ERR_ARG, "batch: mass %d is not finite", l);
        for (int r = 0; r < c.nrhs; ++r) sigma[l * c.nrhs + r] = 4.0 * masses[l] * masses[l];
    }
    return batch_solve_pairs(c, sigma.data(), tol.data(), b, x, prm, stats, caller);
}

ks_status_t batch_solve_pairs(BatchCtx& c, const double* sigma, const double* tol,
                              const double* const* b, double* const* x,
                              const ks_solver_params& prm, ks_batch_stats* stats,
                              hipStream_t caller)
{
    const auto t0 = std::chrono::steady_clock::now();
    const hipStream_t s = enter_stream(c, caller);
    std::vector<double> param(2 * (size_t)c.npairs);
    for (int p = 0; p < c.npairs; ++p) {
        KS_REQUIRE(b[p] && x[p] && b[p] != x[p], KS_ERR_ARG, "batch: bad vectors for pair %d", p);
        KS_REQUIRE(std::isfinite(sigma[p]) && sigma[p] >= 0.0 && tol[p] > 0.0, KS_ERR_ARG,
                   "batch: bad shift or tolerance for pair %d", p);
        param[p] = sigma[p];
        param[c.npairs + p] = tol[p];
    }
    KS_HIP(hipMemcpyAsync(c.pair_param, param.data(), sizeof(double) * param.size(),
                          hipMemcpyHostToDevice, s));
    batch_io(c, c.b64, reinterpret_cast<const void* const*>(b), 1, s);
    batch_io(c, c.x64, reinterpret_cast<const void* const*>(x), 1, s);
    if (c.dx32) KS_HIP(hipMemsetAsync(c.dx32, 0, c.dx32_bytes, s));   // outside any graph
    batch_clock_kernel<<<1, 1, 0, s>>>(c.clock);
    run(c, 3, s);   // |b|^2 tile partials
    batch_init_pairs_kernel<<<c.npairs, kFin, 0, s>>>(c.lats_dev, c.nrhs, c.pairs, c.partials,
                                                      c.pair_param, c.npairs,
                                                      c.prec == KS_F64 ? 0.0 : prm.delta,
                                                      prm.max_iter, c.b2);
    KS_HIP(hipGetLastError());

    // the step sequence (the first step computes the initial residual in FP64), captured once per configuration into a graph of `chunk` steps
    const int chunk = std::max(1, prm.check_every);
    if (!c.graph_exec || c.graph_chunk != chunk) {
        if (c.graph_exec) (void)hipGraphExecDestroy(c.graph_exec);
        c.graph_exec = nullptr;
        hipGraph_t graph;
        KS_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
        try {
            for (int k = 0; k < chunk; ++k) run(c, 0, s);
            batch_census_kernel<<<1, 256, 0, s>>>(c.pairs, c.npairs, c.census);
        } catch (...) {
            hipGraph_t g2;
            (void)hipStreamEndCapture(s, &g2);
            throw;
        }
        KS_HIP(hipStreamEndCapture(s, &graph));
        const hipError_t e = hipGraphInstantiate(&c.graph_exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        KS_HIP(e);
        c.graph_chunk = chunk;
    }
    int max_chunks = prm.max_iter / chunk + 4;
    for (int it = 0; it < max_chunks; ++it) {
        KS_HIP(hipGraphLaunch(c.graph_exec, s));
        KS_HIP(hipMemcpyAsync(c.census_host, c.census, sizeof(int), hipMemcpyDeviceToHost, s));
        KS_HIP(hipStreamSynchronize(s));
        if (*c.census_host >= c.npairs) break;
    }
    KS_HIP(hipMemcpyAsync(c.pairs_host, c.pairs, sizeof(BatchPair) * c.npairs, hipMemcpyDeviceToHost, s));
    unsigned long long start = 0;
    KS_HIP(hipMemcpyAsync(&start, c.clock, sizeof(start), hipMemcpyDeviceToHost, s));
    std::vector<double> b2(c.npairs);
    KS_HIP(hipMemcpyAsync(b2.data(), c.b2, sizeof(double) * c.npairs, hipMemcpyDeviceToHost, s));
    if (c.dx32) run(c, 4, s);   // every pair's remaining FP32 increments into x
    batch_io(c, c.x64, reinterpret_cast<const void* const*>(x), 0, s);
    int dev = 0, khz = 100000;
    KS_HIP(hipGetDevice(&dev));
    if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0)
        khz = 100000;
    ks_status_t result = KS_SUCCESS;
    for (int p = 0; p < c.npairs; ++p) {
        const BatchPair& q = c.pairs_host[p];
        ks_batch_stats& o = stats[p];
        o.iters = q.iter;
        o.reliable_updates = q.ru;
        o.true_rel_resid = b2[p] > 0 ? std::sqrt(q.true_r2 / b2[p]) : 0.0;
        o.seconds = (q.done && q.t_done >= start) ? (double)(q.t_done - start) / (khz * 1e3) : -1.0;
        o.status = q.done ? q.status : KS_ERR_NOT_CONVERGED;
        if (o.status != KS_SUCCESS && result == KS_SUCCESS) result = (ks_status_t)o.status;
    }
    c.last_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    if (result != KS_SUCCESS) set_error("batch: at least one pair failed (first code %d)", (int)result);
    return result;
}

// Autotuner: tile size (64 / 128 / 256 sites per block) and schedule (one block per tile, or
// a persistent grid of k blocks per CU that strides over the tile table), timed on the
// inner-precision multi-RHS Dslash of this batch.
void batch_tune(BatchCtx& c, hipStream_t caller)
{
    const hipStream_t s = enter_stream(c, caller);
    int dev = 0;
    KS_HIP(hipGetDevice(&dev));
    int cus = 256;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 256;
    // every pair active for timing
    for (int p = 0; p < c.npairs; ++p) {
        BatchPair q{};
        c.pairs_host[p] = q;
    }
    KS_HIP(hipMemcpyAsync(c.pairs, c.pairs_host, sizeof(BatchPair) * c.npairs, hipMemcpyHostToDevice, s));
    KS_HIP(hipMemsetAsync(c.ps, 0x3f, c.inner_bytes, s));
    hipEvent_t e0, e1;
    KS_HIP(hipEventCreate(&e0));
    KS_HIP(hipEventCreate(&e1));
    float best = 1e30f;
    int best_k = 0, best_pers = 0;
    for (int k = 0; k < 3; ++k) {
        c.set_tiles(k, s);
        for (int pers : {0, 1, 2, 4, 8}) {
            c.persistent = pers * cus;
            for (int w = 0; w < 2; ++w) run(c, 2, s);
            KS_HIP(hipEventRecord(e0, s));
            for (int w = 0; w < 5; ++w) run(c, 2, s);
            KS_HIP(hipEventRecord(e1, s));
            KS_HIP(hipEventSynchronize(e1));
            float ms = 0.f;
            KS_HIP(hipEventElapsedTime(&ms, e0, e1));
            if (ms < best) {
                best = ms;
                best_k = k;
                best_pers = c.persistent;
            }
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    c.set_tiles(best_k, s);
    c.persistent = best_pers;
    c.tuned_us = best * 1e3f / 5;
}

}  // namespace ks
