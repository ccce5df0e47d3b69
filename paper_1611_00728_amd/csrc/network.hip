// Gauge-covariant preconditioner network on the GPU: forward (inference), adjoint and
// weight-gradient passes, A-norm loss, Adam.
//
// Layer:  y_c(x) = sum_{c', p} w_{c c' p} (T_p phi_{c'})(x), nine paths p: the identity,
// T_{+mu} phi(x) = V_mu(x) phi(x+mu) (p = 1+mu) and T_{-mu} phi(x) = V_mu(x-mu)^+ phi(x-mu)
// (p = 5+mu), with the operator's fat link V.  The network is N = L^+ L, L two free layers
// (1 -> 8 -> 8): it applies four layers 1 -> 8 -> 8 -> 8 -> 1, the last two the adjoints of
// the first two, so N is Hermitian and <v, N v> = |L v|^2 (no activation).
// Activations live on the full lattice as two checkerboard halves, complex FP32.  Here transports
// and channel mixing are FP32 (training, and the FP32 inference path), the mixing of the layers
// with eight outputs and the weight gradients as FP32 matrix-core products; inference also has
// a binary16 form (network_mfma.hip).
//
// The adjoint of a layer, y -> sum_p T_p^+ W_p^H y, is again a layer: channels swapped,
// weights w'_{c' c pbar} = conj(w_{c c' p}), pbar the reversed path (T_{+mu}^+ = T_{-mu}).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "ks_cg_step.h"
#include "ks_device.h"
#include "ks_net.h"
#include "ks_solvers.h"

namespace ks {

namespace {

constexpr int kNT = 256;

// Activations of C channels: [parity][colour][channel pair][Vh] of float4 (two complex channels
// side by side, so that a lane reads 16 bytes) for C = 8, [parity][colour][Vh] of float2 for C = 1.
// Only the even half of a one-channel level is used: the network's input and its output's
// gradient are zero on odd sites, and the odd half of its output is not needed.
__device__ __forceinline__ float4* act_pair(float4* a, int par, int k, int q, int vh)
{
    return a + (size_t)((par * 3 + k) * 4 + q) * vh;
}
__device__ __forceinline__ const float4* act_pair(const float4* a, int par, int k, int q, int vh)
{
    return a + (size_t)((par * 3 + k) * 4 + q) * vh;
}

// even half of a one-channel level, as a vector that a first layer reads
struct ActPlanes {
    using R = float;
    __device__ static __forceinline__ void load(const void* b, int vh, int h, cx<R> v[3])
    {
        const float2* p = static_cast<const float2*>(b);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float2 t = p[(size_t)k * vh + h];
            v[k] = {t.x, t.y};
        }
    }
};

typedef float float4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float4_t mfma4(float a, float b, float4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Layer 8 -> 8 or 1 -> 8.  For 16 sites and one colour the mixing is a real GEMM
// D[16 x 16 sites] += A[16 x 4] B[4 x 16 sites] per step on v_mfma_f32_16x16x4_f32 (FP32 operands
// and sums).  Lane (n, g) of a wave (site n, group g) transports every input channel of its site
// along the two hops of direction mu = g; row g of a B fragment is then one real of the
// transported channel of group g's own path, and the A fragment holds the four paths' weights of
// that channel.  Row 4 q + r of D is channel 2 q + r / 2, its real (r even) or imaginary part, so
// lane (n, q) ends up with the channel pair q of site n: one 16-byte store per colour.
// On the vector ALUs the mixing took three quarters of the layer's 9.2 kflop per site and bound
// it (8 -> 8 layer at 32^4 434 us, 16^3 x 32 57 us, 16^4 35.6 us; now 292, 41, 22).  Per 16 sites 108
// MFMA of 32 cycles and some 900 vector instructions of 4; the two hardly overlap (at 32^4 33 % and
// 34 % of the SIMDs' cycles), and at 32^4 the layer fetches 1.6 GB beyond the L2 (5.9 TB/s with
// its stores).  The A fragments are formed from the weights in LDS once per block; a wave works
// on per_wave groups of 16 consecutive sites, both hops' loads first (two waves per SIMD; three
// or four with fewer loads in flight 10-20 % slower).
template <int CIN, class IN, bool kStream>
__global__ __launch_bounds__(256, CIN == 8 ? 2 : 4) void net_mix_kernel(Geom geo, const void* __restrict__ in,
                                                         float4* __restrict__ out,
                                                         const void* __restrict__ fat_e,
                                                         const void* __restrict__ fat_o,
                                                         const float2* __restrict__ w,
                                                         const double* __restrict__ scale,
                                                         const int* __restrict__ gate, int per_wave)
{
    static_assert(CIN == 8 || CIN == 1, "input channels");
    constexpr int kId = CIN == 8 ? 4 : 1;            // identity fragments
    constexpr int kF = kId + 2 * CIN * 2;            // then (hop j, channel, real / imaginary)
    __shared__ float frag[kF][64];
    if (gate && *gate) return;
    for (int e = threadIdx.x; e < kF * 64; e += 256) {
        const int f = e / 64, l = e % 64;
        const int m = l % 16, k = l / 16;            // A[m][k] sits in lane m + 16 k
        const int co = 2 * (m >> 2) + ((m & 3) >> 1);
        int ci, part, p;
        bool used = true;
        if (f < kId) {
            ci = CIN == 8 ? 2 * k + (f >> 1) : 0;
            part = CIN == 8 ? (f & 1) : (k & 1);
            used = CIN == 8 || k < 2;
            p = 0;
        } else {
            const int q = f - kId;
            part = q & 1;
            ci = (q >> 1) % CIN;
            p = (q >> 1) / CIN ? 5 + k : 1 + k;
        }
        const float2 wc = w[(co * CIN + ci) * 9 + p];
        // Re y = wr ur - wi ui, Im y = wr ui + wi ur; the stored backward links are -V^+
        const float a = ((m & 1) == part) ? wc.x : part ? -wc.y : wc.y;
        frag[f][l] = !used ? 0.f : p >= 5 ? -a : a;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int n = lane & 15, g = lane >> 4;
    const int vh = geo.Vh;
    const float sc = scale ? (float)*scale : 1.f;
    const int wave = xcd_tile(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6);
#pragma unroll 1
    for (int it = 0; it < per_wave; ++it) {
        const int t = (wave * per_wave + it) * 16 + n;
        if (t - n >= 2 * vh) return;
        const bool live = t < 2 * vh;                // a dead lane works on site 0, unstored
        const int par = (live && t >= vh) ? 1 : 0;
        const int h = live ? t - par * vh : 0;
        const void* fat = par ? fat_o : fat_e;
        int c[4];
        cb_coords(geo, h, par, c);
        const int i = site_index(geo, c);
        float4_t acc[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) acc[a] = {0.f, 0.f, 0.f, 0.f};
        if constexpr (CIN == 8) {
            const float4* x = static_cast<const float4*>(in);
            float4 own[3], v[2][4][3];
            cx<float> m[2][9];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int nb = lane_hop(geo, i, c, g, j ? -1 : +1);
                load_link<KS_F32, 9, kStream>(fat, j * 4 + g, geo.lp, h, m[j]);
                if (j == 0) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) own[a] = act_pair(x, par, a, g, vh)[h];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int b = 0; b < 3; ++b) v[j][q][b] = act_pair(x, 1 - par, b, q, vh)[nb];
            }
            __builtin_amdgcn_sched_barrier(0);       // both hops' loads go out first
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                acc[a] = mfma4(frag[0][lane], own[a].x, acc[a]);
                acc[a] = mfma4(frag[1][lane], own[a].y, acc[a]);
                acc[a] = mfma4(frag[2][lane], own[a].z, acc[a]);
                acc[a] = mfma4(frag[3][lane], own[a].w, acc[a]);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
#pragma unroll
                for (int ci = 0; ci < 8; ++ci) {
                    cx<float> u[3];
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        u[a] = {0.f, 0.f};
#pragma unroll
                        for (int b = 0; b < 3; ++b) {
                            const float4 y = v[j][ci >> 1][b];
                            if (ci & 1) cfma(u[a], m[j][a * 3 + b], cx<float>{y.z, y.w});
                            else cfma(u[a], m[j][a * 3 + b], cx<float>{y.x, y.y});
                        }
                    }
                    const int f = kId + (j * 8 + ci) * 2;
#pragma unroll
                    for (int a = 0; a < 3; ++a) acc[a] = mfma4(frag[f][lane], u[a].r, acc[a]);
#pragma unroll
                    for (int a = 0; a < 3; ++a) acc[a] = mfma4(frag[f + 1][lane], u[a].i, acc[a]);
                }
            }
        } else {
            // odd input sites are zero: even outputs take the identity, odd ones the hops
            if (__any(live && par == 0)) {
                cx<typename IN::R> v[3];
                IN::load(in, vh, h, v);
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const float re = sc * (float)v[a].r, im = sc * (float)v[a].i;
                    acc[a] = mfma4(frag[0][lane], par || g > 1 ? 0.f : g ? im : re, acc[a]);
                }
            }
            if (__any(par == 1)) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int nb = lane_hop(geo, i, c, g, j ? -1 : +1);
                    cx<float> m[9], u[3];
                    cx<typename IN::R> v[3];
                    load_link<KS_F32, 9, kStream>(fat, j * 4 + g, geo.lp, h, m);
                    IN::load(in, vh, nb, v);
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        u[a] = {0.f, 0.f};
#pragma unroll
                        for (int b = 0; b < 3; ++b)
                            cfma(u[a], m[a * 3 + b],
                                 cx<float>{sc * (float)v[b].r, sc * (float)v[b].i});
                        acc[a] = mfma4(frag[kId + j * 2][lane], par ? u[a].r : 0.f, acc[a]);
                        acc[a] = mfma4(frag[kId + j * 2 + 1][lane], par ? u[a].i : 0.f, acc[a]);
                    }
                }
            }
        }
        if (live) {
#pragma unroll
            for (int a = 0; a < 3; ++a)
                act_pair(out, par, a, g, vh)[h] = make_float4(acc[a][0], acc[a][1], acc[a][2], acc[a][3]);
        }
    }
}

// The last layer, 8 -> 1, on even sites: four lanes per site, one direction each (lane (n, g) as
// above).  The channels are summed at the neighbour before the transport, one transport per hop
// instead of eight; lane g takes the identity path of channels 2 g and 2 g + 1.
template <class OUT, bool kStream>
__global__ __launch_bounds__(256) void net_last_kernel(Geom geo, const float4* __restrict__ in,
                                                       void* __restrict__ out,
                                                       const void* __restrict__ fat_e,
                                                       const float2* __restrict__ w,
                                                       const double* __restrict__ scale,
                                                       const int* __restrict__ gate)
{
    __shared__ float2 ws[72];
    if (gate && *gate) return;
    if (threadIdx.x < 72) ws[threadIdx.x] = w[threadIdx.x];
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int n = lane & 15, g = lane >> 4;
    const int vh = geo.Vh;
    const int t = xcd_tile(blockIdx.x, gridDim.x) * 64 + (threadIdx.x >> 6) * 16 + n;
    const bool live = t < vh;
    const int h = live ? t : vh - 1;
    int c[4];
    cb_coords(geo, h, 0, c);
    const int i = site_index(geo, c);
    cx<float> y[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float4 v = act_pair(in, 0, a, g, vh)[h];
        const float2 w0 = ws[(2 * g) * 9], w1 = ws[(2 * g + 1) * 9];
        y[a] = {0.f, 0.f};
        cfma(y[a], cx<float>{w0.x, w0.y}, cx<float>{v.x, v.y});
        cfma(y[a], cx<float>{w1.x, w1.y}, cx<float>{v.z, v.w});
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int nb = lane_hop(geo, i, c, g, j ? -1 : +1);
        const int p = j ? 5 + g : 1 + g;
        cx<float> m[9], z[3];
        load_link<KS_F32, 9, kStream>(fat_e, j * 4 + g, geo.lp, h, m);
#pragma unroll
        for (int b = 0; b < 3; ++b) z[b] = {0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float2 w0 = ws[(2 * q) * 9 + p], w1 = ws[(2 * q + 1) * 9 + p];
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const float4 v = act_pair(in, 1, b, q, vh)[nb];
                cfma(z[b], cx<float>{w0.x, w0.y}, cx<float>{v.x, v.y});
                cfma(z[b], cx<float>{w1.x, w1.y}, cx<float>{v.z, v.w});
            }
        }
        const float sg = j ? -1.f : 1.f;             // the store holds -V(x - mu)^+
#pragma unroll
        for (int b = 0; b < 3; ++b) z[b] = {sg * z[b].r, sg * z[b].i};
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) cfma(y[a], m[a * 3 + b], z[b]);
    }
#pragma unroll
    for (int o = 16; o < 64; o *= 2)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            y[a].r += __shfl_xor(y[a].r, o, 64);
            y[a].i += __shfl_xor(y[a].i, o, 64);
        }
    if (live && g == 0) {
        const float inv = (float)(1.0 / (scale ? *scale : 1.0));
        cx<typename OUT::R> v[3];
#pragma unroll
        for (int a = 0; a < 3; ++a)
            v[a] = {(typename OUT::R)(inv * y[a].r), (typename OUT::R)(inv * y[a].i)};
        OUT::store(out, vh, h, v);
    }
}

// Weight gradients G_w[c][c'][p] = sum over sites and colours of conj((T_p phi_c')(x)_a) G_c(x)_a:
// a GEMM over (site, colour) on v_mfma_f32_16x16x4_f32, D[real of G][real of u] += A B with four
// sites of one colour per step.  A block walks tiles of 64 sites; a thread transports one
// channel pair of one site per path (the next path's link and vectors are loaded meanwhile) and
// stages it in LDS in rows of the site's 16 reals, from which the fragments are read; wave w
// takes the products of sites 16 w .. 16 w + 15.  Of its 12 steps per path and tile each
// wgrad_steps start from zero and are added to FP64 registers: 48 products per FP32 sum between
// layers of eight channels, 12 where a layer has one (few values, whose FP64 additions cost
// nothing beside the transports).  The waves' sums are combined in FP64 in a fixed order, and
// the block writes one partial per value.  Against every thread
// multiplying its slice of the sites from LDS for one (c, c'): 8 -> 8 at 16^4 55 -> 25 us, 8 -> 1
// 39 -> 14.5, 1 -> 8 33 -> 8.9.
constexpr int kWTile = 64;
constexpr int kWPitch = 20;                // floats per staged row of 16 (bank spread)
constexpr int kWStage = 3 * kWTile * kWPitch;

// matrix-core steps (of four sites and one colour) per FP32 sum; channels: the fewer of a layer's two
__host__ __device__ constexpr int wgrad_steps(int channels) { return channels == 8 ? 12 : 3; }

// v, or zeros (by component: a choice between two structures would go through scratch memory)
__device__ __forceinline__ float4 keep_if(bool on, float4 v)
{
    return make_float4(on ? v.x : 0.f, on ? v.y : 0.f, on ? v.z : 0.f, on ? v.w : 0.f);
}

// D[r] of a lane: row 4 (lane / 16) + r, column lane % 16
__device__ __forceinline__ void wgrad_spill(double* red, int wave, int lane, const double d[4])
{
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave * 256 + (4 * (lane / 16) + r) * 16 + lane % 16] = d[r];
}

__device__ __forceinline__ double wgrad_sum(const double* red, int row, int col)
{
    double s = 0.0;
#pragma unroll
    for (int wv = 0; wv < 4; ++wv) s += red[wv * 256 + row * 16 + col];
    return s;
}

// the real (reim 0) or imaginary part of sum conj(u) g from the sums of products of reals
__device__ __forceinline__ double wgrad_value(const double* red, int row, int col, int reim)
{
    return reim ? wgrad_sum(red, row + 1, col) - wgrad_sum(red, row, col + 1)
                : wgrad_sum(red, row, col) + wgrad_sum(red, row + 1, col + 1);
}

// 8 -> COUT, the paths 3 y, 3 y + 1, 3 y + 2 of block column y (nine paths' FP64 sums in one block
// hold 236 registers: two waves per SIMD, 26 us for an 8 -> 8 layer at 16^4).  COUT = 1: G lives
// on even sites only.
template <int COUT, bool kStream>
__global__ __launch_bounds__(kNT, 3) void net_wgrad8_kernel(Geom g, const float4* __restrict__ in,
                                                            const void* __restrict__ gy,
                                                            const void* __restrict__ fat_e,
                                                            const void* __restrict__ fat_o,
                                                            double* __restrict__ partials)
{
    __shared__ __align__(16) float us[2][kWStage];
    __shared__ __align__(16) float gs[COUT == 8 ? kWStage : 3 * kWTile * 2];
    const int vh = g.Vh;
    const int nsites = COUT == 8 ? 2 * vh : vh;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, kk = lane >> 4;
    const int p0 = 3 * blockIdx.y;
    double acc[3][4];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[p][r] = 0.0;
    const int ntiles = (nsites + kWTile - 1) / kWTile;
    int buf = 0;
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int t = tile * kWTile + lane;
        const bool live = t < nsites;
        const int par = (live && t >= vh) ? 1 : 0;
        const int h = live ? t - par * vh : 0;
        const void* fat = par ? fat_o : fat_e;
        int c[4];
        cb_coords(g, h, par, c);
        const int i = site_index(g, c);
        // a path's link and input vectors; path 0 is the site itself
        auto fetch = [&](int p, cx<float> m[9], float4 v[3]) {
            const int s = p - 1, mu = s & 3;
            const int d = s >= 4 ? -1 : +1;
            const int cm = (mu == 0 ? c[0] : mu == 1 ? c[1] : mu == 2 ? c[2] : c[3]) + d;
            const int nx = g.n[mu];
            const int nb = (i + (d + (cm < 0 ? nx : 0) - (cm >= nx ? nx : 0)) * g.stride[mu]) >> 1;
            if (p > 0) load_link<KS_F32, 9, kStream>(fat, s, g.lp, h, m);
#pragma unroll
            for (int k = 0; k < 3; ++k)
                v[k] = act_pair(in, p > 0 ? 1 - par : par, k, wave, vh)[p > 0 ? nb : h];
        };
        float4 gv[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if constexpr (COUT == 8) {
                gv[k] = act_pair(static_cast<const float4*>(gy), par, k, wave, vh)[h];
            } else if (wave == k) {
                const float2 v = static_cast<const float2*>(gy)[(size_t)k * vh + h];
                gv[k] = make_float4(v.x, v.y, 0.f, 0.f);
            }
        }
        cx<float> m[9];
        float4 v[3];
        fetch(p0, m, v);
        // gs is read by no wave any more: all have passed the last path's barrier and read their
        // A fragments before it
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if constexpr (COUT == 8)
                *reinterpret_cast<float4*>(&gs[(k * kWTile + lane) * kWPitch + 4 * wave]) =
                    keep_if(live, gv[k]);
            else if (wave == k)
                *reinterpret_cast<float2*>(&gs[(k * kWTile + lane) * 2]) =
                    make_float2(live ? gv[k].x : 0.f, live ? gv[k].y : 0.f);
        }
        float a[12];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int p = p0 + q;
            float4 u[3];
            if (p == 0) {
#pragma unroll
                for (int k = 0; k < 3; ++k) u[k] = v[k];
            } else {
                const float sg = p > 4 ? -1.f : 1.f;  // the store holds -V(x - mu)^+
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    cx<float> x0 = {0.f, 0.f}, x1 = {0.f, 0.f};
#pragma unroll
                    for (int b = 0; b < 3; ++b) {
                        cfma(x0, m[k * 3 + b], cx<float>{v[b].x, v[b].y});
                        cfma(x1, m[k * 3 + b], cx<float>{v[b].z, v[b].w});
                    }
                    u[k] = make_float4(sg * x0.r, sg * x0.i, sg * x1.r, sg * x1.i);
                }
            }
#pragma unroll
            for (int k = 0; k < 3; ++k)
                *reinterpret_cast<float4*>(&us[buf][(k * kWTile + lane) * kWPitch + 4 * wave]) =
                    keep_if(live, u[k]);
            if (q < 2) fetch(p + 1, m, v);
            __syncthreads();
            if (q == 0) {
#pragma unroll
                for (int s = 0; s < 12; ++s) {
                    const int row = (s % 3) * kWTile + 16 * wave + 4 * (s / 3) + kk;
                    if constexpr (COUT == 8) a[s] = gs[row * kWPitch + n];
                    else a[s] = n < 2 ? gs[row * 2 + n] : 0.f;
                }
            }
            float4_t d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 12; ++s) {
                const int row = (s % 3) * kWTile + 16 * wave + 4 * (s / 3) + kk;
                d = mfma4(a[s], us[buf][row * kWPitch + n], d);
                if ((s + 1) % wgrad_steps(COUT) == 0) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[q][r] += (double)d[r];
                    d = {0.f, 0.f, 0.f, 0.f};
                }
            }
            buf ^= 1;
        }
    }
    constexpr int NV = COUT * 8 * 9 * 2;
    double* red = reinterpret_cast<double*>(&us[0][0]);   // the staged rows are done with
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        __syncthreads();
        wgrad_spill(red, wave, lane, acc[q]);
        __syncthreads();
        for (int e = tid; e < COUT * 16; e += kNT) {
            const int reim = e & 1, ci = (e >> 1) % 8, co = e / 16;
            partials[(size_t)blockIdx.x * NV + ((co * 8 + ci) * 9 + p0 + q) * 2 + reim] +=
                wgrad_value(red, 2 * co, 2 * ci, reim);
        }
    }
}

// 1 -> 8.  phi lives on even sites only: the identity path takes even sites, and the eight hops
// take odd ones, all eight in one product (column 2 (p - 1) + real / imaginary part).
template <bool kStream>
__global__ __launch_bounds__(kNT) void net_wgrad1_kernel(Geom g, const float2* __restrict__ in,
                                                         const float4* __restrict__ gy,
                                                         const void* __restrict__ fat_o,
                                                         double* __restrict__ partials)
{
    __shared__ __align__(16) float us[kWStage];
    __shared__ __align__(16) float gs[kWStage];
    __shared__ double red[4 * 256];
    const int vh = g.Vh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, kk = lane >> 4;
    double acc[2][4];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[q][r] = 0.0;
    const int half = (vh + kWTile - 1) / kWTile;
    for (int tile = blockIdx.x; tile < 2 * half; tile += gridDim.x) {
        const int par = tile >= half ? 1 : 0;        // the same for the whole tile
        const int t = (tile - par * half) * kWTile + lane;
        const bool live = t < vh;
        const int h = live ? t : 0;
        float4 gv[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) gv[k] = act_pair(gy, par, k, wave, vh)[h];
        cx<float> u[2][3];                           // par 1: the two hops along mu = wave
        if (par) {
            int c[4];
            cb_coords(g, h, 1, c);
            const int i = site_index(g, c);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int nb = lane_hop(g, i, c, wave, j ? -1 : +1);
                cx<float> m[9], v[3];
                load_link<KS_F32, 9, kStream>(fat_o, j * 4 + wave, g.lp, h, m);
                ActPlanes::load(in, vh, nb, v);
                const float sg = j ? -1.f : 1.f;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    cx<float> x = {0.f, 0.f};
#pragma unroll
                    for (int b = 0; b < 3; ++b) cfma(x, m[k * 3 + b], v[b]);
                    u[j][k] = {sg * x.r, sg * x.i};
                }
            }
        } else {
            cx<float> v[3];
            ActPlanes::load(in, vh, h, v);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                u[0][k] = {wave == 0 ? v[k].r : 0.f, wave == 0 ? v[k].i : 0.f};
                u[1][k] = {0.f, 0.f};
            }
        }
        __syncthreads();                             // the last tile's products are done
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            float* ur = &us[(k * kWTile + lane) * kWPitch];
            // columns 2 mu (forward) and 8 + 2 mu (backward) of the hops
#pragma unroll
            for (int j = 0; j < 2; ++j)
                *reinterpret_cast<float2*>(ur + 8 * j + 2 * wave) =
                    make_float2(live ? u[j][k].r : 0.f, live ? u[j][k].i : 0.f);
            *reinterpret_cast<float4*>(&gs[(k * kWTile + lane) * kWPitch + 4 * wave]) =
                keep_if(live, gv[k]);
        }
        __syncthreads();
        float4_t d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 12; ++s) {
            const int row = (s % 3) * kWTile + 16 * wave + 4 * (s / 3) + kk;
            d = mfma4(gs[row * kWPitch + n], us[row * kWPitch + n], d);
            if ((s + 1) % wgrad_steps(1) == 0) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    acc[0][r] += par ? 0.0 : (double)d[r];
                    acc[1][r] += par ? (double)d[r] : 0.0;
                }
                d = {0.f, 0.f, 0.f, 0.f};
            }
        }
    }
    constexpr int NV = 8 * 9 * 2;
    for (int q = 0; q < 2; ++q) {
        __syncthreads();
        wgrad_spill(red, wave, lane, q ? acc[1] : acc[0]);
        __syncthreads();
        const int np = q ? 8 : 1;
        for (int e = tid; e < 8 * np * 2; e += kNT) {
            const int reim = e & 1, p = (e >> 1) % np, co = (e >> 1) / np;
            partials[(size_t)blockIdx.x * NV + (co * 9 + (q ? p + 1 : 0)) * 2 + reim] +=
                wgrad_value(red, 2 * co, 2 * p, reim);
        }
    }
}

// grad[k] = sum_b partials[b][k] for 16 values per block: slice j of a value's 64 threads adds
// partials j, j + 64, ..., then the slices in a fixed order.  (64 values and 16 slices per block
// leave the 512 x 1152 partials of an 8 -> 8 layer to 18 CUs: 11.1 us.)
__global__ __launch_bounds__(1024) void net_grad_finish_kernel(const double* __restrict__ partials,
                                                               int nblocks, int nv,
                                                               double* __restrict__ grad)
{
    __shared__ double red[16][16];
    const int l = threadIdx.x & 15, j = threadIdx.x >> 4;
    const int k = blockIdx.x * 16 + l;               // nv is a multiple of 16
    double s = 0.0;
#pragma unroll 4
    for (int b = j; b < nblocks; b += 64) s += partials[(size_t)b * nv + k];
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    if ((threadIdx.x & 63) < 16) red[threadIdx.x >> 6][l] = s;
    __syncthreads();
    if (threadIdx.x < 16) {
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < 16; ++q) v += red[q][l];
        grad[k] = v;
    }
}

// w'[c'][c][pbar] = conj(w[c][c'][p])
__global__ void net_adjoint_weights_kernel(const float2* __restrict__ w, float2* __restrict__ wa,
                                           int cin, int cout)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= cin * cout * 9) return;
    const int p = k % 9, ci = (k / 9) % cin, o = k / (9 * cin);
    const int pb = p == 0 ? 0 : (p <= 4 ? p + 4 : p - 4);
    const float2 v = w[k];
    wa[(ci * cout + o) * 9 + pb] = make_float2(v.x, -v.y);
}

// One pair's x and b (complex128 [Vh][3]): the even sites of the network's input b, and partials of
// x^+ A x = Re<x, b>
__global__ __launch_bounds__(kNT) void net_pair_kernel(int vh, const double2* __restrict__ x,
                                                       const double2* __restrict__ b,
                                                       float2* __restrict__ act,
                                                       double* __restrict__ partials)
{
    const int h = blockIdx.x * kNT + threadIdx.x;
    double s = 0.0;
    if (h < vh)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double2 u = x[(size_t)h * 3 + k], v = b[(size_t)h * 3 + k];
            s += u.x * v.x + u.y * v.y;
            act[(size_t)k * vh + h] = make_float2((float)v.x, (float)v.y);
        }
    s = block_sum<kNT>(s);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// A-norm loss term of one pair and the output gradient: with y = N(b) and ay = A y (FP64 planes, even
// sites), x^+ A x from the partials xax_part (as many as blocks here), partial sums of Re<y - x, A y - b> = (y - x)^+ A (y - x)
// (A x = b) and G = 2 (A y - b) / (x^+ A x npairs) on even sites (the Wirtinger gradient of the
// pair's loss is 2 A (y - x) over its normalisation).
__global__ __launch_bounds__(kNT) void net_anorm_loss_kernel(int vh, const double2* __restrict__ y,
                                                             const double2* __restrict__ ay,
                                                             const double2* __restrict__ b,
                                                             const double2* __restrict__ x,
                                                             const double* __restrict__ xax_part,
                                                             int npairs, float2* __restrict__ gy,
                                                             double* __restrict__ partials)
{
    const int h = blockIdx.x * kNT + threadIdx.x;
    const double xax = fused_total<kNT>(fused_load<kNT>(xax_part, gridDim.x));
    double s = 0.0;
    if (h < vh) {
        const double coef = 2.0 / (xax * npairs);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double2 o = y[(size_t)k * vh + h];
            const double2 a = ay[(size_t)k * vh + h];
            const double2 bv = b[(size_t)h * 3 + k];
            const double2 xv = x[(size_t)h * 3 + k];
            const double rr = a.x - bv.x, ri = a.y - bv.y;
            s += (o.x - xv.x) * rr + (o.y - xv.y) * ri;
            gy[(size_t)k * vh + h] = make_float2((float)(coef * rr), (float)(coef * ri));
        }
    }
    s = block_sum<kNT>(s);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// Sums of a chunk of pairs: block 2 k the partials of x^+ A x of pair k, block 2 k + 1 those of its
// loss, lists of n[k] partials at a pitch of `pitch`.
constexpr int kPairChunk = 32;

struct PairCounts {
    int n[kPairChunk];
};

__global__ __launch_bounds__(kNT) void net_pair_sums_kernel(const double* __restrict__ partials,
                                                            int pitch, PairCounts c,
                                                            double* __restrict__ out)
{
    const double s = fused_total<kNT>(
        fused_load<kNT>(partials + (size_t)blockIdx.x * pitch, c.n[blockIdx.x / 2]));
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

__device__ __forceinline__ int reversed_path(int p) { return p == 0 ? 0 : (p <= 4 ? p + 4 : p - 4); }

// FP32 weights of the four applied layers from the FP64 free weights: layers 1 and 2 as they
// are, layer 3 = adjoint of layer 2, layer 4 = adjoint of layer 1
// (w'[c'][c][pbar] = conj(w[c][c'][p])).
__global__ void net_expand_kernel(const double2* __restrict__ w, float2* __restrict__ w32)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    constexpr int n1 = 8 * 1 * 9, n2 = 8 * 8 * 9;
    if (k >= kNetLayerWeights) return;
    double2 v;
    if (k < n1 + n2) {
        v = w[k];
    } else if (k < n1 + 2 * n2) {
        const int j = k - n1 - n2;                        // layer 3: [c'][c][q], 8 x 8
        const int q = j % 9, c = (j / 9) % 8, cp = j / 72;
        const double2 u = w[n1 + (c * 8 + cp) * 9 + reversed_path(q)];
        v = make_double2(u.x, -u.y);
    } else {
        const int j = k - n1 - 2 * n2;                    // layer 4: [0][c][q]
        const int q = j % 9, c = j / 9;
        const double2 u = w[c * 9 + reversed_path(q)];
        v = make_double2(u.x, -u.y);
    }
    w32[k] = make_float2((float)v.x, (float)v.y);
}

// Gradient of the free weights from the four layers' gradients: a free weight collects its
// own layer's G plus the conjugate of G at its place in the adjoint layer.
__global__ void net_fold_kernel(const double2* __restrict__ g4, double2* __restrict__ g)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    constexpr int n1 = 8 * 1 * 9, n2 = 8 * 8 * 9;
    if (k >= kNetWeights) return;
    double2 a = g4[k], t;
    if (k < n1) {                                          // w1[c][0][p]
        const int p = k % 9, c = k / 9;
        t = g4[n1 + 2 * n2 + c * 9 + reversed_path(p)];    // layer 4 [0][c][pbar]
    } else {                                               // w2[c][c'][p]
        const int j = k - n1;
        const int p = j % 9, cp = (j / 9) % 8, c = j / 72;
        t = g4[n1 + n2 + (cp * 8 + c) * 9 + reversed_path(p)];   // layer 3 [c'][c][pbar]
    }
    g[k] = make_double2(a.x + t.x, a.y - t.y);
}

// One Adam step on every real of the FP64 master weights.
__global__ void net_adam_kernel(double* __restrict__ w, double* __restrict__ m,
                                double* __restrict__ v, const double* __restrict__ grad, int n,
                                double lr, double b1, double b2, double eps, double c1, double c2)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const double gk = grad[k];
    const double mk = b1 * m[k] + (1.0 - b1) * gk;
    const double vk = b2 * v[k] + (1.0 - b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    const double mh = mk / c1, vhat = vk / c2;
    w[k] = w[k] - lr * mh / (sqrt(vhat) + eps);
}

// The fat FP32 links of both parities up to this size are read through the caches: the
// last-level one (256 MB) then still holds them, beside the activations, for the next layer.
constexpr size_t kCachedLinks = (size_t)100 << 20;
bool links_cached(const Geom& G) { return (size_t)2 * 8 * 9 * 8 * G.lp <= kCachedLinks; }

// 1 -> 8 (IN: the vector the layer reads, times *scale) or 8 -> 8 (IN = void)
template <int CIN, class IN>
void mix_layer(ks_gauge_t g, const void* in, float2* out, const float2* w, hipStream_t s,
               const double* scale = nullptr, const int* gate = nullptr)
{
    const LinkStore& st = g->store[KS_F32][0];
    const Geom& G = g->geom;
    // consecutive groups per wave: 512 blocks (the two per CU that are resident at a time) on small
    // lattices, 1024 on large ones (8 -> 8 layer, 512 / 1024 blocks: 16^4 22.1 / 24.8 us, 32^4
    // 322 / 293 us)
    const int groups = blocks_for(2L * G.Vh, 16);
    const int per_wave = blocks_for(groups, 4 * (groups <= 16384 ? 512 : 1024));
    const int nb = blocks_for(groups, 4 * per_wave);
    float4* o = reinterpret_cast<float4*>(out);
    if (links_cached(G))
        net_mix_kernel<CIN, IN, false><<<nb, 256, 0, s>>>(G, in, o, st.fat[0], st.fat[1], w, scale,
                                                          gate, per_wave);
    else
        net_mix_kernel<CIN, IN, true><<<nb, 256, 0, s>>>(G, in, o, st.fat[0], st.fat[1], w, scale,
                                                         gate, per_wave);
    KS_HIP(hipGetLastError());
}

template <class OUT>
void last_layer(ks_gauge_t g, const float2* in, void* out, const float2* w, hipStream_t s,
                const double* scale = nullptr, const int* gate = nullptr)
{
    const LinkStore& st = g->store[KS_F32][0];
    const Geom& G = g->geom;
    const int nb = blocks_for(G.Vh, 64);
    const float4* x = reinterpret_cast<const float4*>(in);
    if (links_cached(G))
        net_last_kernel<OUT, false><<<nb, 256, 0, s>>>(G, x, out, st.fat[0], w, scale, gate);
    else
        net_last_kernel<OUT, true><<<nb, 256, 0, s>>>(G, x, out, st.fat[0], w, scale, gate);
    KS_HIP(hipGetLastError());
}

void expand_weights(NetCtx& n, hipStream_t s)
{
    net_expand_kernel<<<blocks_for(kNetLayerWeights, 256), 256, 0, s>>>(
        reinterpret_cast<const double2*>(n.w64), reinterpret_cast<float2*>(n.w32));
    KS_HIP(hipGetLastError());
}

// 256 blocks times three path columns, the three per CU that are resident at a time (8 -> 8 layer,
// 256 / 512 blocks: 16^4 25.1 / 28.5 us, 32^4 425 / 462 us; the 1 -> 8 layer's 101 / 137 us)
constexpr int kWgrad8Blocks = 256;

// Blocks of a layer's weight-gradient kernel on a lattice.
int wgrad_blocks(int cin, int cout, const Geom& G)
{
    const int tiles = cin == 1 ? 2 * blocks_for(G.Vh, kWTile)
                               : blocks_for(cout == 8 ? 2L * G.Vh : G.Vh, kWTile);
    return std::min(tiles, cin == 1 ? kWgradBlocks : kWgrad8Blocks);
}

// Adds the pair's weight gradient to each block's sums in `part`: the blocks' sums run over all
// pairs and are added up once (a finishing launch per pair and layer was 23 us of a pair's 261 at 16^4).
template <int CIN, int COUT>
void wgrad(ks_gauge_t g, const float2* in, const float2* gy, double* part, hipStream_t s)
{
    const LinkStore& st = g->store[KS_F32][0];
    const Geom& G = g->geom;
    const int nb = wgrad_blocks(CIN, COUT, G);
    const bool cached = links_cached(G);
    if constexpr (CIN == 1) {
        const float4* g4 = reinterpret_cast<const float4*>(gy);
        if (cached) net_wgrad1_kernel<false><<<nb, kNT, 0, s>>>(G, in, g4, st.fat[1], part);
        else net_wgrad1_kernel<true><<<nb, kNT, 0, s>>>(G, in, g4, st.fat[1], part);
    } else {
        const float4* x = reinterpret_cast<const float4*>(in);
        if (cached)
            net_wgrad8_kernel<COUT, false><<<dim3(nb, 3), kNT, 0, s>>>(G, x, gy, st.fat[0], st.fat[1], part);
        else
            net_wgrad8_kernel<COUT, true><<<dim3(nb, 3), kNT, 0, s>>>(G, x, gy, st.fat[0], st.fat[1], part);
    }
    KS_HIP(hipGetLastError());
}

// the four layers from the vector IN at `in` to the vector OUT at `out`
template <class IN, class OUT>
void forward(NetCtx& n, NetBuffers& B, ks_gauge_t g, const void* in, void* out, hipStream_t s,
             const double* scale = nullptr, const int* gate = nullptr)
{
    const float2* w = reinterpret_cast<const float2*>(n.w32);
    mix_layer<1, IN>(g, in, B.act[1], w + layer_weight_offset(0), s, scale, gate);
    mix_layer<8, void>(g, B.act[1], B.act[2], w + layer_weight_offset(1), s, nullptr, gate);
    mix_layer<8, void>(g, B.act[2], B.act[3], w + layer_weight_offset(2), s, nullptr, gate);
    last_layer<OUT>(g, B.act[3], out, w + layer_weight_offset(3), s, scale, gate);
}

}  // namespace

const int kLayerIn[4] = {1, 8, 8, 8};

double net_model_bytes(int use_mfma, double vec_bytes)
{
    if (use_mfma) return 2.0 * net_mfma_model_bytes_per_site(vec_bytes);
    // per even site: the first layer reads the even input vector and the odd site's eight FP32
    // links and writes both sites' activations, the middle two read and write every site's and
    // read all links, the last reads both sites' activations and the even site's links and writes
    // the even output vector
    const double links = 8 * 72.0, act = 8 * 24.0;
    const double first = vec_bytes + links + 2 * act, middle = 2 * (act + links + act);
    return first + 2 * middle + 2 * act + links + vec_bytes;
}
const int kLayerOut[4] = {8, 8, 8, 1};

size_t layer_weight_offset(int l)
{
    size_t o = 0;
    for (int k = 0; k < l; ++k) o += (size_t)kLayerIn[k] * kLayerOut[k] * 9;
    return o;
}

NetBuffers& net_buffers(NetCtx& n, const Geom& g)
{
    NetBuffers& B = n.bufs[g.Vh];
    if (B.vh == 0) {
        const size_t half = (size_t)3 * g.Vh * sizeof(float2);   // one channel, one parity
        alloc_once(B.act[0], half);
        alloc_once(B.grad[4], half);
        for (int l = 1; l < 4; ++l) {
            alloc_once(B.act[l], half * 16);
            alloc_once(B.grad[l], half * 16);
        }
        B.vh = g.Vh;
    }
    return B;
}

void net_free(NetCtx* n)
{
    if (!n) return;
    for (auto& kv : n->bufs) {
        for (int l = 0; l < 5; ++l) {
            device_free(kv.second.act[l]);
            device_free(kv.second.grad[l]);
            device_free(kv.second.act16[l]);
        }
    }
    device_free(n->w64);
    device_free(n->w32);
    device_free(n->wadj);
    device_free(n->adam_m);
    device_free(n->adam_v);
    device_free(n->grad);
    device_free(n->grad4);
    device_free(n->scal);
    device_free(n->part);
    device_free(n->wmma);
    if (n->host) (void)hipHostFree(n->host);
    delete n;
}

NetCtx* net_create(const double* w_host)
{
    NetCtx* n = new NetCtx();
    try {
        const size_t nr = 2 * (size_t)kNetWeights;
        const size_t nl = 2 * (size_t)kNetLayerWeights;
        n->w64 = static_cast<double*>(device_alloc(sizeof(double) * nr));
        n->w32 = static_cast<float*>(device_alloc(sizeof(float) * nl));
        n->wadj = static_cast<float*>(device_alloc(sizeof(float) * nl));
        n->adam_m = static_cast<double*>(device_alloc(sizeof(double) * nr));
        n->adam_v = static_cast<double*>(device_alloc(sizeof(double) * nr));
        n->grad = static_cast<double*>(device_alloc(sizeof(double) * nr));
        n->grad4 = static_cast<double*>(device_alloc(sizeof(double) * nl));
        n->scal = static_cast<double*>(device_alloc(sizeof(double) * 64));
        KS_HIP(hipHostMalloc(reinterpret_cast<void**>(&n->host), sizeof(double) * 64));
        net_set_weights(*n, w_host, nullptr);
    } catch (...) {
        net_free(n);
        throw;
    }
    return n;
}

void net_set_weights(NetCtx& n, const double* w_host, hipStream_t s)
{
    const int nr = 2 * kNetWeights;
    KS_HIP(hipMemcpyAsync(n.w64, w_host, sizeof(double) * nr, hipMemcpyHostToDevice, s));
    KS_HIP(hipMemsetAsync(n.adam_m, 0, sizeof(double) * nr, s));
    KS_HIP(hipMemsetAsync(n.adam_v, 0, sizeof(double) * nr, s));
    expand_weights(n, s);
    KS_HIP(hipStreamSynchronize(s));
    n.step = 0;
    n.version += 1;
}

void net_get_weights(NetCtx& n, double* w_host, hipStream_t s)
{
    KS_HIP(hipMemcpyAsync(w_host, n.w64, sizeof(double) * 2 * kNetWeights, hipMemcpyDeviceToHost, s));
    KS_HIP(hipStreamSynchronize(s));
}

void net_get_state(NetCtx& n, double* w, double* m, double* v, int* step, hipStream_t s)
{
    const size_t nb = sizeof(double) * 2 * kNetWeights;
    KS_HIP(hipMemcpyAsync(w, n.w64, nb, hipMemcpyDeviceToHost, s));
    KS_HIP(hipMemcpyAsync(m, n.adam_m, nb, hipMemcpyDeviceToHost, s));
    KS_HIP(hipMemcpyAsync(v, n.adam_v, nb, hipMemcpyDeviceToHost, s));
    KS_HIP(hipStreamSynchronize(s));
    *step = n.step;
}

void net_set_state(NetCtx& n, const double* w, const double* m, const double* v, int step,
                   hipStream_t s)
{
    const size_t nb = sizeof(double) * 2 * kNetWeights;
    KS_HIP(hipMemcpyAsync(n.w64, w, nb, hipMemcpyHostToDevice, s));
    KS_HIP(hipMemcpyAsync(n.adam_m, m, nb, hipMemcpyHostToDevice, s));
    KS_HIP(hipMemcpyAsync(n.adam_v, v, nb, hipMemcpyHostToDevice, s));
    expand_weights(n, s);
    KS_HIP(hipStreamSynchronize(s));
    n.step = step;
    n.version += 1;
}

// out_dev = N(in_dev) (complex128 [Vh][3], even sites); FP32 transports and mixing.
void net_apply_f32(NetCtx& n, ks_gauge_t g, const double* in, double* out, hipStream_t s)
{
    gauge_prepare(g, KS_F32, KS_RECON_18, s);
    forward<SpinorAos, SpinorAos>(n, net_buffers(n, g->geom), g, in, out, s);
}

void net_apply_spinor(NetCtx& n, ks_gauge_t g, ks_prec_t prec, const void* r, void* z,
                      const double* in_scale, const int* gate, int use_mfma, hipStream_t s)
{
    KS_REQUIRE(prec == KS_F64 || prec == KS_F32, KS_ERR_ARG,
               "network: the solver's vectors must be FP64 or FP32");
    if (use_mfma) {
        net_apply_mfma_spinor(n, g, prec, r, z, in_scale, gate, s);
        return;
    }
    gauge_prepare(g, KS_F32, KS_RECON_18, s);
    NetBuffers& B = net_buffers(n, g->geom);
    if (prec == KS_F64)
        forward<Spinor<KS_F64>, Spinor<KS_F64>>(n, B, g, r, z, s, in_scale, gate);
    else
        forward<Spinor<KS_F32>, Spinor<KS_F32>>(n, B, g, r, z, s, in_scale, gate);
}

// A-norm loss of the pairs and its gradient: the four applied layers' gradients, summed over the
// pairs, go to n.grad4 and fold into the free weights' gradient n.grad.
double net_loss_grad(NetCtx& n, int npairs, const ks_gauge_t* gauges, const double* sigma,
                     const double* const* b, const double* const* x, hipStream_t s)
{
    // n.part: per layer the blocks' weight gradients (cleared here), then for each pair of a chunk
    // the partials of x^+ A x and of its loss
    int blocks[4] = {0, 0, 0, 0}, pitch = 0;
    for (int j = 0; j < npairs; ++j) {
        const Geom& G = gauges[j]->geom;
        for (int l = 0; l < 4; ++l)
            blocks[l] = std::max(blocks[l], wgrad_blocks(kLayerIn[l], kLayerOut[l], G));
        pitch = std::max(pitch, blocks_for(G.Vh, kNT));
    }
    size_t at[5] = {0};
    int nv[4];
    for (int l = 0; l < 4; ++l) {
        nv[l] = kLayerIn[l] * kLayerOut[l] * 9 * 2;
        at[l + 1] = at[l] + (size_t)blocks[l] * nv[l];
    }
    const size_t need = at[4] + (size_t)std::min(npairs, kPairChunk) * 2 * pitch;
    if (n.part_size < need) {
        device_free(n.part);
        n.part = nullptr;
        n.part_size = 0;
        n.part = static_cast<double*>(device_alloc(sizeof(double) * need));
        n.part_size = need;
    }
    double* pair_part = n.part + at[4];
    KS_HIP(hipMemsetAsync(n.part, 0, sizeof(double) * at[4], s));
    const float2* w = reinterpret_cast<const float2*>(n.w32);
    float2* wa = reinterpret_cast<float2*>(n.wadj);
    for (int l = 1; l < 4; ++l) {
        const size_t o = layer_weight_offset(l);
        net_adjoint_weights_kernel<<<blocks_for(kLayerIn[l] * kLayerOut[l] * 9, 256), 256, 0, s>>>(
            w + o, wa + o, kLayerIn[l], kLayerOut[l]);
    }
    KS_HIP(hipGetLastError());
    // x^+ A x and the loss of a pair stay on the device while its kernels are queued; the host
    // reads those of up to kPairChunk pairs together (reading each when it was needed left the GPU
    // idle twice per pair, some 35 us)
    double loss = 0.0;
    PairCounts counts{};
    for (int j = 0; j < npairs; ++j) {
        const int c = j % kPairChunk;
        ks_gauge_t g = gauges[j];
        gauge_prepare(g, KS_F32, KS_RECON_18, s);
        Workspace& ws = workspace(g);
        NetBuffers& B = net_buffers(n, g->geom);
        const int vh = g->geom.Vh;
        const int nb = blocks_for(vh, kNT);
        counts.n[c] = nb;
        double* xax = pair_part + (size_t)2 * c * pitch;
        const double2* bj = reinterpret_cast<const double2*>(b[j]);
        const double2* xj = reinterpret_cast<const double2*>(x[j]);
        net_pair_kernel<<<nb, kNT, 0, s>>>(vh, xj, bj, B.act[0], xax);
        // y = N(b), written as FP64 planes for A y in FP64 on the pair's lattice
        forward<ActPlanes, Spinor<KS_F64>>(n, B, g, B.act[0], ws.r64, s);
        apply_A64(g, sigma[j], ws.r64, ws.ax64, s, nullptr);
        net_anorm_loss_kernel<<<nb, kNT, 0, s>>>(vh, reinterpret_cast<const double2*>(ws.r64),
                                                 reinterpret_cast<const double2*>(ws.ax64), bj, xj,
                                                 xax, npairs, B.grad[4], xax + pitch);
        KS_HIP(hipGetLastError());
        // backward: weight gradients and the adjoint layers
        wgrad<8, 1>(g, B.act[3], B.grad[4], n.part + at[3], s);
        mix_layer<1, ActPlanes>(g, B.grad[4], B.grad[3], wa + layer_weight_offset(3), s);
        wgrad<8, 8>(g, B.act[2], B.grad[3], n.part + at[2], s);
        mix_layer<8, void>(g, B.grad[3], B.grad[2], wa + layer_weight_offset(2), s);
        wgrad<8, 8>(g, B.act[1], B.grad[2], n.part + at[1], s);
        mix_layer<8, void>(g, B.grad[2], B.grad[1], wa + layer_weight_offset(1), s);
        wgrad<1, 8>(g, B.act[0], B.grad[1], n.part + at[0], s);
        if (c == kPairChunk - 1 || j == npairs - 1) {
            net_pair_sums_kernel<<<2 * (c + 1), kNT, 0, s>>>(pair_part, pitch, counts, n.scal);
            KS_HIP(hipGetLastError());
            KS_HIP(hipMemcpyAsync(n.host, n.scal, sizeof(double) * 2 * (c + 1),
                                  hipMemcpyDeviceToHost, s));
            KS_HIP(hipStreamSynchronize(s));
            for (int k = 0; k <= c; ++k) {
                const double q = n.host[2 * k];
                KS_REQUIRE(q > 0, KS_ERR_ARG, "network training: pair %d has Re<x, b> <= 0",
                           j - c + k);
                loss += n.host[2 * k + 1] / (q * npairs);
            }
        }
    }
    for (int l = 0; l < 4; ++l)
        net_grad_finish_kernel<<<nv[l] / 16, 1024, 0, s>>>(n.part + at[l], blocks[l], nv[l],
                                                           n.grad4 + 2 * layer_weight_offset(l));
    net_fold_kernel<<<blocks_for(kNetWeights, 256), 256, 0, s>>>(
        reinterpret_cast<const double2*>(n.grad4), reinterpret_cast<double2*>(n.grad));
    KS_HIP(hipGetLastError());
    return loss;
}

void net_adam(NetCtx& n, double lr, hipStream_t s)
{
    const int nr = 2 * kNetWeights;
    n.step += 1;
    const double b1 = 0.9, b2 = 0.999;
    net_adam_kernel<<<blocks_for(nr, 256), 256, 0, s>>>(n.w64, n.adam_m, n.adam_v, n.grad, nr, lr,
                                                       b1, b2, 1e-8, 1.0 - std::pow(b1, n.step),
                                                       1.0 - std::pow(b2, n.step));
    KS_HIP(hipGetLastError());
    expand_weights(n, s);
    n.version += 1;
}

}  // namespace ks
