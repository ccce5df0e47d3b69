// Link derivative ("force") of the multi-shift pseudofermion action
//     S = sum_i r_i phi^+ (sigma_i - D_eo D_oe)^-1 phi
// from the shifted solutions X_i = (sigma_i - D_eo D_oe)^-1 phi, the quantity the multi-mass
// solver's output feeds in molecular-dynamics evolution (the fermion force of Sec. 5's outlook).
// With Y_i = D_oe X_i and Psi_i = X_i on even sites, Y_i on odd sites, a change of the links
// changes S by sum_{x,mu} 2 Re Tr[dV_mu(x) FV_mu(x) + dW_mu(x) FW_mu(x)] with
//     FV_mu(x) = eps(x) sum_i r_i Psi_i(x+mu) Psi_i(x)^+,
//     FW_mu(x) = eps(x) sum_i r_i Psi_i(x+3mu) Psi_i(x)^+,      eps = +1 even, -1 odd sites.
// The Y_i come from a multi-vector FP64 hopping term (links read once for up to ten X_i);
// one pass over (direction, site) pairs then builds both outer-product sums in registers and
// writes them in the canonical link layout.
#include <algorithm>
#include <vector>

#include "ks_blas.h"
#include "ks_device.h"
#include "ks_solvers.h"

namespace ks {

namespace {

constexpr int kMaxTerms = 32;
constexpr int kTile = 64;               // sites

// The n vectors of one parity: [tiles of 64 sites][n terms][3 colours][64] complex, so that all that
// a neighbourhood of sites holds is one run of memory.  (As 3 n planes of Vh sites each, at a pitch
// that is a multiple of the caches' way size, the rows of a neighbourhood fell on the same sets.)
struct TermVecs {
    double2* p;
    int n;
    __device__ __forceinline__ double2* at(int h) const
    {
        return p + (size_t)(h / kTile) * (n * 3 * kTile) + h % kTile;
    }
};

__device__ __forceinline__ void load_psi(const double2* site, int term, cx<double> v[3])
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double2 t = site[(term * 3 + k) * kTile];
        v[k] = {t.x, t.y};
    }
}

struct TermPtrs {
    const double2* x[kMaxTerms];
    double r[kMaxTerms];
};

// caller's vectors [Vh][3], one per blockIdx.y
__global__ __launch_bounds__(kBlock) void force_import_kernel(int vh, TermPtrs t, TermVecs x)
{
    const int h = blockIdx.x * kBlock + threadIdx.x;
    if (h >= vh) return;
    const double2* src = t.x[blockIdx.y] + (size_t)3 * h;
    double2* dst = x.at(h) + blockIdx.y * (3 * kTile);
#pragma unroll
    for (int k = 0; k < 3; ++k) dst[k * kTile] = src[k];
}

// y_k = D_{par} x_k for the terms [first, last) at once (FP64, 18-real, 8-way links of the output
// parity): each of a site's 16 link matrices is read once for all of them.  Two lanes per output
// site, the halves of a wave: with one group of K terms a half takes the one-link or the Naik
// matrices and a shuffle adds them; with two groups a half takes K terms, which serves up to ten
// with the accumulators of five, the second half's link loads being hits of the same instruction.
// Bound by the vectors that the gathers bring to L2 again and again: two blocks per CU (dynamic
// LDS, and registers for all loads of a hop) keep the span of sites in flight short.  Nine terms,
// 32^3x48: 1010 us in passes of five and four from planes of Vh sites; 780 in one.  Links through the
// caches 850, three blocks per CU 860, four lanes per site by hops 800-910, four groups of three
// terms 860-1010.  Ten terms 1875 us for the whole force, 2230 in two passes of five.
constexpr int kSites = 32;              // per wave
constexpr int kMultiMax = 10;           // terms per pass
constexpr int kMultiLds = 80000;        // of a CU's 160 KB

template <int K, int kGroups>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) void
dslash_multi_kernel(Geom g, int par, const void* __restrict__ fat, const void* __restrict__ naik,
                    TermVecs in, TermVecs out, int first, int last, float fat_scale,
                    float naik_scale)
{
    extern __shared__ double2 one_link[];   // kMultiLds bytes: a thread's own 3 K entries
    static_assert(3 * K * kBlock * sizeof(double2) <= kMultiLds, "one_link");
    const int vh = g.Vh;
    const int wave = xcd_tile(blockIdx.x, gridDim.x) * (kBlock / 64) + (threadIdx.x >> 6);
    const int hh = wave * kSites + threadIdx.x % kSites;
    const int part = (threadIdx.x & 63) / kSites;
    const int t0 = first + (kGroups == 2 ? part * K : 0);
    const int s0 = kGroups == 2 ? 0 : part * 8;
    const bool live = hh < vh;
    const int h = live ? hh : vh - 1;       // a dead lane shadows a live site (no store)
    int c[4];
    cb_coords(g, h, par, c);
    const int i = site_index(g, c);
    cx<double> res[K][3];
#pragma unroll
    for (int q = 0; q < K; ++q)
#pragma unroll
        for (int a = 0; a < 3; ++a) res[q][a] = {0.0, 0.0};
#pragma unroll 1
    for (int u = 0; u < 8 * kGroups; ++u) {
        const int s = s0 + u;
        // slots 0-3: +mu, 4-7: -mu, 8-15: the Naik ones; backward slots hold the negated adjoint
        const int nb = hop_cb(g, i, c, s & 3, (s & 8 ? 3 : 1) * (s & 4 ? -1 : 1));
        const double sc = s & 8 ? (double)naik_scale : (double)fat_scale;
        cx<double> m[9];
        load_link<KS_F64, 9>(s & 8 ? naik : fat, s & 7, g.lp, h, m);
        const double2* site = in.at(nb);
#pragma unroll
        for (int q = 0; q < K; ++q) {
            cx<double> v[3];
            load_psi(site, min(t0 + q, last - 1), v);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                cx<double> u = {0.0, 0.0};
#pragma unroll
                for (int b = 0; b < 3; ++b) cfma(u, m[a * 3 + b], v[b]);
                res[q][a].r = fma(sc, u.r, res[q][a].r);
                res[q][a].i = fma(sc, u.i, res[q][a].i);
            }
        }
        if (kGroups == 2 && u == 7) {
            // the one-link sums wait in LDS, so that the Naik ones start from zero: eight additions
            // to each, as with one group, and the same bits
#pragma unroll
            for (int q = 0; q < K; ++q)
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    one_link[(q * 3 + a) * kBlock + threadIdx.x] = make_double2(res[q][a].r, res[q][a].i);
                    res[q][a] = {0.0, 0.0};
                }
        }
    }
    if constexpr (kGroups == 2) {
#pragma unroll
        for (int q = 0; q < K; ++q)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const double2 f = one_link[(q * 3 + a) * kBlock + threadIdx.x];
                res[q][a].r += f.x;
                res[q][a].i += f.y;
            }
    }
    if constexpr (kGroups == 1) {
#pragma unroll
        for (int q = 0; q < K; ++q)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                res[q][a].r += __shfl_xor(res[q][a].r, 32, 64);
                res[q][a].i += __shfl_xor(res[q][a].i, 32, 64);
            }
    }
    if (!live || (kGroups == 1 && part)) return;
    double2* o = out.at(h);
#pragma unroll
    for (int q = 0; q < K; ++q) {
        if (t0 + q >= last) break;
#pragma unroll
        for (int a = 0; a < 3; ++a)
            o[((t0 + q) * 3 + a) * kTile] = make_double2(res[q][a].r, res[q][a].i);
    }
}

template <int K, int kGroups>
void launch_multi_k(const Geom& G, const LinkStore& st, TermVecs in, TermVecs out, int first,
                    int last, hipStream_t s)
{
    if constexpr (K > 1) {
        if (last - first <= kGroups * (K - 1)) {
            launch_multi_k<K - 1, kGroups>(G, st, in, out, first, last, s);
            return;
        }
    }
    dslash_multi_kernel<K, kGroups><<<blocks_for(2L * G.Vh), kBlock, kMultiLds, s>>>(
        G, 1, st.fat[1], st.naik[1], in, out, first, last, st.fat_scale, st.naik_scale);
    KS_HIP(hipGetLastError());
}

// One block: kOuterSites consecutive lexicographic sites x the four directions (wave w takes
// mu = w), so the four waves that read a site's vectors share them through one CU's L1; blocks
// are remapped so that each XCD walks one contiguous range of sites.  Thread (mu, x) writes
// link t = mu V + x.  The lower half of a wave takes the even sites of the block's pairs of x
// neighbours, the upper half the odd ones, so that each half reads one run of memory (sites in x
// order alternate between the two parities' fields, which doubles the cache accesses: 32^3x48, nine
// terms, 1016 -> 860 us).  The next term's loads ahead of this one's products: no gain (156
// registers, three waves per SIMD).
constexpr int kOuterSites = 64;

__global__ __launch_bounds__(4 * kOuterSites) __attribute__((amdgpu_waves_per_eu(4, 4))) void
force_outer_kernel(Geom g, TermPtrs terms, TermVecs even, TermVecs odd, double2* __restrict__ fv,
                   double2* __restrict__ fw)
{
    const int mu = threadIdx.x / kOuterSites;
    const int lane = threadIdx.x % kOuterSites;
    const long x0 = (long)xcd_tile(blockIdx.x, gridDim.x) * kOuterSites;
    const bool full = x0 + kOuterSites <= g.V;   // uniform over the block
    const int par = lane >> 5;
    const long xe = x0 + 2 * (lane & 31);
    if (!full && xe >= g.V) return;               // only in a ragged last block
    int x = (int)xe;
    int c[4];
    int r = x;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        c[d] = r % g.n[d];
        r /= g.n[d];
    }
    c[3] = r;
    const int up = (c[0] + c[1] + c[2] + c[3] + par) & 1;   // the pair's site of parity par
    x += up;
    c[0] += up;
    const long t = (long)mu * g.V + x;
    const int h = x >> 1;
    const int n1 = hop_cb(g, x, c, mu, +1);
    const int n3 = hop_cb(g, x, c, mu, +3);
    cx<double> a1[9], a3[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        a1[e] = {0.0, 0.0};
        a3[e] = {0.0, 0.0};
    }
    const double2* s0 = (par ? odd : even).at(h);
    const double2* s1 = (par ? even : odd).at(n1);
    const double2* s3 = (par ? even : odd).at(n3);
    for (int i = 0; i < even.n; ++i) {
        cx<double> p0[3], p1[3], p3[3];
        load_psi(s0, i, p0);
        load_psi(s1, i, p1);
        load_psi(s3, i, p3);
        const double ri = terms.r[i];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const cx<double> u1 = {ri * p1[a].r, ri * p1[a].i};
            const cx<double> u3 = {ri * p3[a].r, ri * p3[a].i};
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                // u conj(p0_b)
                a1[a * 3 + b].r = fma(u1.r, p0[b].r, fma(u1.i, p0[b].i, a1[a * 3 + b].r));
                a1[a * 3 + b].i = fma(u1.i, p0[b].r, fma(-u1.r, p0[b].i, a1[a * 3 + b].i));
                a3[a * 3 + b].r = fma(u3.r, p0[b].r, fma(u3.i, p0[b].i, a3[a * 3 + b].r));
                a3[a * 3 + b].i = fma(u3.i, p0[b].r, fma(-u3.r, p0[b].i, a3[a * 3 + b].i));
            }
        }
    }
    const double eps = par ? -1.0 : 1.0;
    if (full) {
        // stage each wave's 64 consecutive links in LDS, then store them as one contiguous,
        // streamed run (a lane's own 144 bytes at a 144-byte lane stride, stored directly,
        // measured slower; streamed without staging, far slower)
        __shared__ dvec2 stage[4][kOuterSites * 9];
        dvec2* sw = stage[mu];
        dvec2* o1 = reinterpret_cast<dvec2*>(fv + ((size_t)mu * g.V + x0) * 9);
        dvec2* o3 = reinterpret_cast<dvec2*>(fw + ((size_t)mu * g.V + x0) * 9);
#pragma unroll
        for (int e = 0; e < 9; ++e) sw[(int)(x - x0) * 9 + e] = dvec2{eps * a1[e].r, eps * a1[e].i};
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 9; ++k)
            __builtin_nontemporal_store(sw[k * kOuterSites + lane], o1 + k * kOuterSites + lane);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 9; ++e) sw[(int)(x - x0) * 9 + e] = dvec2{eps * a3[e].r, eps * a3[e].i};
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 9; ++k)
            __builtin_nontemporal_store(sw[k * kOuterSites + lane], o3 + k * kOuterSites + lane);
        return;
    }
    double2* o1 = fv + (size_t)t * 9;
    double2* o3 = fw + (size_t)t * 9;
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        o1[e] = make_double2(eps * a1[e].r, eps * a1[e].i);
        o3[e] = make_double2(eps * a3[e].r, eps * a3[e].i);
    }
}

}  // namespace

int force_max_terms() { return kMaxTerms; }

void force_core(ks_gauge_t g, int nterm, const double* residues, const double* const* x_even,
                double* force_fat, double* force_naik, hipStream_t s)
{
    Workspace& w = workspace(g);
    const Geom& G = g->geom;
    if (w.force_terms < nterm) {
        const size_t ab = (size_t)blocks_for(G.Vh, kTile) * kTile * 3 * sizeof(double2);
        for (double*& v : w.force_psi) {
            device_free(v);
            v = nullptr;
        }
        w.bytes -= 2 * ab * w.force_terms;
        w.force_terms = 0;
        for (double*& v : w.force_psi) v = static_cast<double*>(device_alloc(ab * nterm));
        w.force_terms = nterm;
        w.bytes += 2 * ab * nterm;
    }
    const TermVecs even{reinterpret_cast<double2*>(w.force_psi[0]), nterm};
    const TermVecs odd{reinterpret_cast<double2*>(w.force_psi[1]), nterm};
    TermPtrs terms{};
    for (int i = 0; i < nterm; ++i) {
        terms.x[i] = reinterpret_cast<const double2*>(x_even[i]);
        terms.r[i] = residues[i];
    }
    force_import_kernel<<<dim3(blocks_for(G.Vh), nterm), kBlock, 0, s>>>(G.Vh, terms, even);
    KS_HIP(hipGetLastError());
    // Y_i = D_oe X_i, up to kMultiMax terms per pass over the odd sites' links, in even shares
    const LinkStore& st = g->store[KS_F64][recon_index(KS_RECON_18)];
    if (!st.ready) gauge_prepare(g, KS_F64, KS_RECON_18, s);
    const int passes = (nterm + kMultiMax - 1) / kMultiMax;
    for (int k = 0; k < passes; ++k) {
        const int a = nterm * k / passes, b = nterm * (k + 1) / passes;
        // up to five terms the halves of a wave share one group's matrices (five, 32^3x48: 1180 us
        // for the whole force against 1204 with two groups, where 1.5 times the loads serve six)
        if (b - a <= kMultiMax / 2) launch_multi_k<kMultiMax / 2, 1>(G, st, even, odd, a, b, s);
        else launch_multi_k<kMultiMax / 2, 2>(G, st, even, odd, a, b, s);
    }
    force_outer_kernel<<<(unsigned)((G.V + kOuterSites - 1) / kOuterSites), 4 * kOuterSites, 0, s>>>(
        G, terms, even, odd, reinterpret_cast<double2*>(force_fat), reinterpret_cast<double2*>(force_naik));
    KS_HIP(hipGetLastError());
}

}  // namespace ks
