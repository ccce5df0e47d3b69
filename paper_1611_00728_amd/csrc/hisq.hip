// Fat and Naik links built from thin links on the device: a two-level smearing with a unitary
// projection in between (the HISQ construction that produces the links the solver of Sec. 3
// reads).  All fields are FP64 in the link layout of ks_gauge_load, [4][V][3][3] complex with
// lexicographic sites.
//
// Staple of a field M on mu-links in the signed transverse direction (nu, s):
//     S[M](x) = L(x) M(x + s nu) L(x + mu)^+,   L(y) = U_nu(y) (s = +1), U_nu(y - nu)^+ (s = -1).
// A smearing with coefficients (c1, c3, c5, c7, cL) is
//     F_mu = c1 U + cL sum_a S_a[S_a[U]] + sum_a S_a[ c3 U + sum_b S_b[ c5 U + c7 sum_c S_c[U] ] ]
// over signed transverse directions on distinct axes (6 three-link, 24 five-link, 48
// seven-link staples, 6 double-width Lepage staples; the nesting follows from linearity of the
// staple in M).  A middle field depends on the axes left over only, not on the sign of the outer
// direction, so per mu three fields of each kind are enough:
//     T_n = c5 U + c7 (S_{+n}[U] + S_{-n}[U]),
//     I_l = c3 U + sum over the two axes m off mu and l of (S_{+m} + S_{-m})[T_n], n the third,
//     F   = c1 U + sum_l (S_{+l} + S_{-l})[I_l] + cL sum_a S_a[S_a[U]],
// three passes of 6, 12 and 6 staples (the Lepage staples are formed again in the last).  Building
// every middle field in registers at the outer staple's end instead takes 6 + 24 + 6 staples and
// twelve launches per mu: 30.3 ms for both smearings at 32^4, 7.5 ms in three passes.
// The passes run two waves per SIMD and are bound by the matrices they fetch beyond the XCD's L2
// (five-link pass 11.8 GB in 1.55 ms in plain order, 7.6 TB/s; see smear_place).
#include <map>
#include <mutex>

#include "ks_device.h"

namespace ks {

namespace {

using cxd = cx<double>;

struct Mat {
    cxd e[9];
};

__device__ __forceinline__ Mat load_mat(const double2* f, long site)
{
    Mat m;
    const double2* p = f + site * 9;
#pragma unroll
    for (int k = 0; k < 9; ++k) m.e[k] = {p[k].x, p[k].y};
    return m;
}

__device__ __forceinline__ void store_mat(double2* f, long site, const Mat& m)
{
    double2* p = f + site * 9;
#pragma unroll
    for (int k = 0; k < 9; ++k) p[k] = make_double2(m.e[k].r, m.e[k].i);
}

__device__ __forceinline__ Mat mul(const Mat& a, const Mat& b)
{
    Mat c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cxd s = {0.0, 0.0};
#pragma unroll
            for (int k = 0; k < 3; ++k) cfma(s, a.e[i * 3 + k], b.e[k * 3 + j]);
            c.e[i * 3 + j] = s;
        }
    return c;
}

__device__ __forceinline__ void site_coords(const Geom& g, long x, int c[4])
{
    long r = x;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        c[d] = (int)(r % g.n[d]);
        r /= g.n[d];
    }
    c[3] = (int)r;
}

// Scratch fields hold one direction's links tile after tile of 64 sites, entry-major within a
// tile ([x / 64][9][64]), so that a wave's loads of one entry are a contiguous kilobyte.
constexpr int kTileSites = 64;
inline long tile_sites(long vol) { return (vol + kTileSites - 1) / kTileSites * kTileSites; }

// byte offset of a site's first entry within a field
__device__ __forceinline__ size_t tile_off(int site)
{
    return ((size_t)((unsigned)site / kTileSites) * (9 * kTileSites) + (unsigned)site % kTileSites) *
           sizeof(double2);
}

__device__ __forceinline__ Mat load_tiled(const double2* f, int site)
{
    const size_t o = tile_off(site);
    Mat m;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const char* fk = reinterpret_cast<const char*>(f + k * kTileSites);
        const double2 v = *reinterpret_cast<const double2*>(fk + o);
        m.e[k] = {v.x, v.y};
    }
    return m;
}

// streamed: the fields a pass writes are read by the next one only, and would push the fields
// that its neighbours still read out of the L2 (32^4, all passes: 9.0 -> 8.8 ms)
__device__ __forceinline__ void store_tiled(double2* f, int site, const Mat& m)
{
    const size_t o = tile_off(site);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        char* fk = reinterpret_cast<char*>(f + k * kTileSites);
        __builtin_nontemporal_store(dvec2{m.e[k].r, m.e[k].i}, reinterpret_cast<dvec2*>(fk + o));
    }
}

__device__ __forceinline__ void axpy_mat(Mat& acc, double w, const Mat& m)
{
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        acc.e[k].r = fma(w, m.e[k].r, acc.e[k].r);
        acc.e[k].i = fma(w, m.e[k].i, acc.e[k].i);
    }
}

// acc += w a m b^+ (the staple of the middle link m in a positive direction).  The staple is summed
// up by itself and rounded into acc once: acc is several times its size, and six products per real
// entry added to acc one by one round at that size six times (level 2 alone, random links: relative
// error 2.8e-16, 1.3e-16 this way; both smearings at 32^4 7.41 and 7.43 ms).
__device__ __forceinline__ void staple_fwd(Mat& acc, const Mat& a, const Mat& m, const Mat& b,
                                           double w = 1.0)
{
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        cxd t[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            t[j] = {0.0, 0.0};
#pragma unroll
            for (int k = 0; k < 3; ++k) cfma(t[j], a.e[i * 3 + k], m.e[k * 3 + j]);
            t[j] = {w * t[j].r, w * t[j].i};
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cxd s = {0.0, 0.0};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const cxd y = b.e[j * 3 + k];
                s.r = fma(t[k].r, y.r, fma(t[k].i, y.i, s.r));
                s.i = fma(t[k].i, y.r, fma(-t[k].r, y.i, s.i));
            }
            acc.e[i * 3 + j].r += s.r;
            acc.e[i * 3 + j].i += s.i;
        }
    }
}

// acc += w a^+ m b (in a negative direction)
__device__ __forceinline__ void staple_bwd(Mat& acc, const Mat& a, const Mat& m, const Mat& b,
                                           double w = 1.0)
{
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        cxd t[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            t[j] = {0.0, 0.0};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const cxd x = a.e[k * 3 + i], y = m.e[k * 3 + j];
                t[j].r = fma(x.r, y.r, fma(x.i, y.i, t[j].r));
                t[j].i = fma(x.r, y.i, fma(-x.i, y.r, t[j].i));
            }
            t[j] = {w * t[j].r, w * t[j].i};
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cxd s = {0.0, 0.0};
#pragma unroll
            for (int k = 0; k < 3; ++k) cfma(s, t[k], b.e[k * 3 + j]);
            acc.e[i * 3 + j].r += s.r;
            acc.e[i * 3 + j].i += s.i;
        }
    }
}

__device__ __forceinline__ Mat zero_mat()
{
    Mat m;
#pragma unroll
    for (int k = 0; k < 9; ++k) m.e[k] = {0.0, 0.0};
    return m;
}

// Offsets of a site's neighbours along an axis.  They add up over different axes, since a wrap
// depends on its own axis' coordinate only.
__device__ __forceinline__ int step_of(const Geom& g, const int c[4], int d, int k)
{
    const int cm = c[d] + k, n = g.n[d];
    return (k + (cm < 0 ? n : 0) - (cm >= n ? n : 0)) * g.stride[d];
}

// v[0..2]: the values of the three axes other than mu (uniform), in order; returns mu's value
__device__ __forceinline__ int off_axes(const int a[4], int mu, int v[3])
{
    v[0] = mu == 0 ? a[1] : a[0];
    v[1] = mu <= 1 ? a[2] : a[1];
    v[2] = mu <= 2 ? a[3] : a[2];
    return mu < 2 ? (mu == 0 ? a[0] : a[1]) : (mu == 2 ? a[2] : a[3]);
}

// The fields of one smearing pass: U the four directions' links (`field` double2 each); T and I
// three scratch fields for each direction of the pass (mu0, ...).  pb, zb: the order of the
// tiles, see smear_place.
struct SmearArgs {
    const double2* U;
    double2* T;
    double2* I;
    size_t field;
    double c1, c3, c5, c7, cl;
    int mu0, pb, zb;
};

// A wave works on a tile of 64 sites and one direction.  f, b (f2, b2): offsets of the neighbours
// one (two) steps along the three axes off mu; fm: one step along mu.
struct Place {
    int x, mu, fm;
    int f[3], b[3], f2[3], b2[3];
    int c[4];
};

// kMus = 4: a block is one tile times the four directions, so its waves share the sites' thin
// links through the CU's L1; kMus = 1: four tiles in the direction mu0.  Each XCD takes one
// contiguous range of tiles of this order: pb tiles of a (z, t) plane times zb planes in z, t after
// t, then the next such column (pb = 0: the tiles as they are numbered).  A column's z and t
// neighbours are then read again while they are in the XCD's L2; the passes are bound by what
// they fetch beyond it (five-link pass at 32^4: 9.9 GB fetched of 2.4 GB of fields in plain
// order, 1.55 -> 1.31 ms with columns of 4 tiles x 4 planes; 2 x 4 1.39, 8 x 4 1.41, 4 x 8 1.40,
// 16 x 4 1.50 ms).
template <int kMus>
__device__ __forceinline__ bool smear_place(const Geom& g, const SmearArgs& t, Place& p)
{
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
    int tile = xcd_tile(blockIdx.x, gridDim.x);
    if (kMus == 1) tile = 4 * tile + w;
    p.mu = kMus == 1 ? t.mu0 : w;
    if ((long)tile * kTileSites >= g.V) return false;
    if (t.pb > 0) {
        const int plane = g.n[0] * g.n[1] / kTileSites;
        int q = tile;
        const int pl = q % t.pb;
        q /= t.pb;
        const int zl = q % t.zb;
        q /= t.zb;
        const int tt = q % g.n[3];
        q /= g.n[3];
        const int pc = q % (plane / t.pb), zc = q / (plane / t.pb);
        tile = (tt * g.n[2] + zc * t.zb + zl) * plane + pc * t.pb + pl;
    }
    p.x = tile * kTileSites + (int)threadIdx.x % kTileSites;
    if (p.x >= g.V) return false;
    int r = p.x;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        p.c[d] = r % g.n[d];
        r /= g.n[d];
    }
    p.c[3] = r;
    int a[4][4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        a[0][d] = step_of(g, p.c, d, 1);
        a[1][d] = step_of(g, p.c, d, -1);
        a[2][d] = step_of(g, p.c, d, 2);
        a[3][d] = step_of(g, p.c, d, -2);
    }
    p.fm = off_axes(a[0], p.mu, p.f);
    (void)off_axes(a[1], p.mu, p.b);
    (void)off_axes(a[2], p.mu, p.f2);
    (void)off_axes(a[3], p.mu, p.b2);
    return true;
}

// the axis of place j off mu
__device__ __forceinline__ int other_axis(int mu, int j) { return j < mu ? j : j + 1; }

// Keeps the loads of one staple after the arithmetic of the one before it: two waves per SIMD
// (192-256 registers) without spills, the best occupancy measured (three: 1.19 instead of 1.05 ms
// for the three-link pass, 1.00 instead of 0.94 for the outer one).
__device__ __forceinline__ void staple_fence() { asm volatile("" ::: "memory"); }

// T_n = c5 U + c7 (S_{+n}[U] + S_{-n}[U]) for the three axes n off mu
template <int kMus>
__global__ __launch_bounds__(256, 2) void smear_three_kernel(Geom g, SmearArgs t)
{
    Place p;
    if (!smear_place<kMus>(g, t, p)) return;
    const double2* Umu = t.U + p.mu * t.field;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const double2* Un = t.U + other_axis(p.mu, j) * t.field;
        const int xf = p.x + p.f[j], xb = p.x + p.b[j];
        Mat s = zero_mat();
        staple_fwd(s, load_tiled(Un, p.x), load_tiled(Umu, xf),
                   load_tiled(Un, p.x + p.fm));
        staple_fence();
        staple_bwd(s, load_tiled(Un, xb), load_tiled(Umu, xb),
                   load_tiled(Un, xb + p.fm));
        staple_fence();
        const Mat u = load_tiled(Umu, p.x);
        Mat o;
#pragma unroll
        for (int k = 0; k < 9; ++k)
            o.e[k] = {fma(t.c7, s.e[k].r, t.c5 * u.e[k].r), fma(t.c7, s.e[k].i, t.c5 * u.e[k].i)};
        store_tiled(t.T + (3 * (p.mu - t.mu0) + j) * t.field, p.x, o);
        staple_fence();
    }
}

// I_l = c3 U + sum over the axes m off mu and l of (S_{+m} + S_{-m})[T_n], n the remaining axis
template <int kMus>
__global__ __launch_bounds__(256, 2) void smear_five_kernel(Geom g, SmearArgs t)
{
    Place p;
    if (!smear_place<kMus>(g, t, p)) return;
    const double2* Umu = t.U + p.mu * t.field;
    const double2* T = t.T + 3 * (p.mu - t.mu0) * t.field;
    Mat in[3];
    {
        const Mat u = load_tiled(Umu, p.x);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            in[j] = zero_mat();
            axpy_mat(in[j], t.c3, u);
        }
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int j1 = (j + 1) % 3, j2 = (j + 2) % 3;
        const double2* Un = t.U + other_axis(p.mu, j) * t.field;
        const int xf = p.x + p.f[j], xb = p.x + p.b[j];
        staple_fence();
        {
            const Mat A = load_tiled(Un, p.x), B = load_tiled(Un, p.x + p.fm);
            staple_fwd(in[j1], A, load_tiled(T + j2 * t.field, xf), B);
            staple_fence();
            staple_fwd(in[j2], A, load_tiled(T + j1 * t.field, xf), B);
        }
        staple_fence();
        {
            const Mat A = load_tiled(Un, xb), B = load_tiled(Un, xb + p.fm);
            staple_bwd(in[j1], A, load_tiled(T + j2 * t.field, xb), B);
            staple_fence();
            staple_bwd(in[j2], A, load_tiled(T + j1 * t.field, xb), B);
        }
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) store_tiled(t.I + (3 * (p.mu - t.mu0) + j) * t.field, p.x, in[j]);
}

// sign of the staggered phase eta_mu and the antiperiodic time boundary on a link of `hops` steps
__device__ __forceinline__ double link_sign(const Geom& g, const int c[4], int mu, int hops)
{
    int e = 0;
    if (mu >= 1) e += c[0];
    if (mu >= 2) e += c[1];
    if (mu >= 3) e += c[2];
    if (mu == 3 && c[3] + hops >= g.n[3]) e += 1;
    return (e & 1) ? -1.0 : 1.0;
}

// F = c1 U + sum_l (S_{+l} + S_{-l})[I_l] + cL (S_{+l}[S_{+l}[U]] + S_{-l}[S_{-l}[U]]).
// kFinal: the sign of the staggered phase and the time boundary is multiplied in and F goes to
// `out` in the layout of ks_gauge_load; otherwise F goes to scratch fields.
template <int kMus, bool kFinal, bool kLepage>
__global__ __launch_bounds__(256, 2) void smear_outer_kernel(
    Geom g, SmearArgs t, double2* __restrict__ out)
{
    Place p;
    if (!smear_place<kMus>(g, t, p)) return;
    const double2* Umu = t.U + p.mu * t.field;
    const double2* I = t.I + 3 * (p.mu - t.mu0) * t.field;
    Mat o = zero_mat();
    axpy_mat(o, t.c1, load_tiled(Umu, p.x));
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const double2* Un = t.U + other_axis(p.mu, j) * t.field;
        const int xf = p.x + p.f[j], xb = p.x + p.b[j];
        staple_fence();
        {
            Mat m = load_tiled(I + j * t.field, xf);
            if constexpr (kLepage) {
                staple_fwd(m, load_tiled(Un, xf), load_tiled(Umu, p.x + p.f2[j]),
                           load_tiled(Un, xf + p.fm), t.cl);
                staple_fence();
            }
            staple_fwd(o, load_tiled(Un, p.x), m, load_tiled(Un, p.x + p.fm));
        }
        staple_fence();
        {
            Mat m = load_tiled(I + j * t.field, xb);
            if constexpr (kLepage) {
                const int z = p.x + p.b2[j];
                staple_bwd(m, load_tiled(Un, z), load_tiled(Umu, z),
                           load_tiled(Un, z + p.fm), t.cl);
                staple_fence();
            }
            staple_bwd(o, load_tiled(Un, xb), m, load_tiled(Un, xb + p.fm));
        }
    }
    if constexpr (kFinal) {
        const double sg = link_sign(g, p.c, p.mu, 1);
#pragma unroll
        for (int k = 0; k < 9; ++k) o.e[k] = {sg * o.e[k].r, sg * o.e[k].i};
        store_mat(out, (long)p.mu * g.V + p.x, o);
    } else {
        store_tiled(out + p.mu * t.field, p.x, o);
    }
}

// links in the layout of ks_gauge_load -> four scratch fields
__global__ __launch_bounds__(256) void tile_links_kernel(int vol, const double2* __restrict__ in,
                                                         double2* __restrict__ out, size_t field)
{
    const int x = blockIdx.x * 256 + threadIdx.x;
    if (x >= vol) return;
    const int mu = blockIdx.y;
    store_tiled(out + mu * field, x, load_mat(in, (long)mu * vol + x));
}

// W = V (V^+ V)^(-1/2) in place, by the scaled Newton iteration for the polar factor,
// X <- (g X + (g X)^-+ ) / 2 with g = |det X|^(-1/3) (1 once that is within 1e-3 of it), at most
// kPolarIters steps; a singular or non-finite V sets *bad.  The iteration converges quadratically
// and ends at a step that moved X by rounding only.  (X^-1)^+ = conj(cof X) det X / |det X|^2, cof
// the cofactors; every entry is divided for itself, by one reciprocal and a residual step each: a
// common factor's rounding turns the whole matrix, and three such matrices make a Naik link
// (relative error of smooth links' W and Naik links, extended precision: 1.20e-16 and 2.52e-16 with
// det X / |det X|^2 as one factor and a last step less, 1.11e-16 and 2.26e-16 this way; 32^4, all:
// 7.51 and 7.54 ms, 7.75 with eighteen divisions).
constexpr int kPolarIters = 40;

__global__ __launch_bounds__(kBlock) void u3_project_kernel(int vol, double2* __restrict__ V,
                                                            size_t field, int* __restrict__ bad)
{
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= vol) return;
    double2* Vmu = V + blockIdx.y * field;
    Mat X = load_tiled(Vmu, x);
    bool ok = true;
    for (int it = 0; it < kPolarIters; ++it) {
        Mat cf;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const int a1 = (a + 1) % 3, a2 = (a + 2) % 3, b1 = (b + 1) % 3, b2 = (b + 2) % 3;
                cxd t = cmul(X.e[a1 * 3 + b1], X.e[a2 * 3 + b2]);
                const cxd u = X.e[a1 * 3 + b2];
                cfma(t, {-u.r, -u.i}, X.e[a2 * 3 + b1]);
                cf.e[a * 3 + b] = t;
            }
        cxd det = {0.0, 0.0};
#pragma unroll
        for (int b = 0; b < 3; ++b) cfma(det, X.e[b], cf.e[b]);
        const double d2 = det.r * det.r + det.i * det.i;
        const double ad = sqrt(d2);
        if (!(ad > 0.0) || !isfinite(ad)) {
            ok = false;
            break;
        }
        const double gam = it < 6 && fabs(ad - 1.0) > 1e-3 ? cbrt(1.0 / ad) : 1.0;
        const double dg = d2 * gam, rd = 1.0 / dg;
        auto over_dg = [&](double v) {
            const double q = v * rd;
            return fma(fma(-q, dg, v), rd, q);
        };
        double diff = 0.0, nrm = 0.0;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const cxd p = cmul({cf.e[k].r, -cf.e[k].i}, det);
            const cxd y = {0.5 * fma(gam, X.e[k].r, over_dg(p.r)),
                           0.5 * fma(gam, X.e[k].i, over_dg(p.i))};
            const double dr = y.r - X.e[k].r, di = y.i - X.e[k].i;
            diff += dr * dr + di * di;
            nrm += y.r * y.r + y.i * y.i;
            X.e[k] = y;
        }
        if (diff <= 1e-30 * nrm) break;
    }
    if (!ok) {
        *bad = 1;
        X = zero_mat();
    }
    store_tiled(Vmu, x, X);
}

// N_mu(x) = c W_mu(x) W_mu(x + mu) W_mu(x + 2 mu) times the staggered phase and the time-boundary
// sign, all four directions
__global__ __launch_bounds__(kBlock) void naik_kernel(Geom g, const double2* __restrict__ W,
                                                      size_t field, double c,
                                                      double2* __restrict__ N)
{
    const int x = xcd_tile(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (x >= g.V) return;
    const int mu = blockIdx.y;
    int cc[4];
    site_coords(g, x, cc);
    const double2* Wm = W + mu * field;
    const int x1 = x + step_of(g, cc, mu, 1), x2 = x + step_of(g, cc, mu, 2);
    Mat r = mul(mul(load_tiled(Wm, x), load_tiled(Wm, x1)), load_tiled(Wm, x2));
    const double s = c * link_sign(g, cc, mu, 3);
#pragma unroll
    for (int k = 0; k < 9; ++k) r.e[k] = {s * r.e[k].r, s * r.e[k].i};
    store_mat(N, (long)mu * g.V + x, r);
}

// F(U; c) of all four directions, kMus of them per pass
template <int kMus, bool kFinal>
void smear(const Geom& G, SmearArgs t, double2* out, hipStream_t st)
{
    const int nb = blocks_for(blocks_for(G.V, kTileSites), 4 / kMus);
    for (t.mu0 = 0; t.mu0 < 4; t.mu0 += kMus) {
        smear_three_kernel<kMus><<<nb, 256, 0, st>>>(G, t);
        smear_five_kernel<kMus><<<nb, 256, 0, st>>>(G, t);
        if (t.cl != 0.0)
            smear_outer_kernel<kMus, kFinal, true><<<nb, 256, 0, st>>>(G, t, out);
        else
            smear_outer_kernel<kMus, kFinal, false><<<nb, 256, 0, st>>>(G, t, out);
        KS_HIP(hipGetLastError());
    }
}

// the largest divisor of n up to `most`
int divisor_upto(int n, int most)
{
    for (int k = most; k > 1; --k)
        if (n % k == 0) return k;
    return 1;
}

}  // namespace

const double kHisqLevel1[5] = {1.0 / 8, 1.0 / 16, 1.0 / 64, 1.0 / 384, 0.0};
const double kHisqLevel2[5] = {1.0, 1.0 / 16, 1.0 / 64, 1.0 / 384, -1.0 / 8};
const double kHisqNaik = -1.0 / 24;

namespace {

// Scratch of the link construction (the tiled thin links, the level-1 links, and per direction
// of a pass three fields T and three I: 32 link fields with all four directions in one pass, 14
// where the device has no room for those), kept per device between calls and grown when a larger
// lattice comes, so that repeated calls allocate nothing.
//
// All four directions share a pass (32 fields) up to this size, a ninth of the card's memory
// (48^3 x 64 takes 30.4 GiB); larger lattices take a direction per pass (32^4: 9.6 ms instead of
// 7.5), so that they need no more memory than their 14 fields.
constexpr size_t kWideScratch = (size_t)32 << 30;

struct HisqScratch {
    void* ptr = nullptr;
    size_t bytes = 0;
};
std::mutex g_hisq_mu;
std::map<int, HisqScratch> g_hisq;

// `bytes` of scratch, or `fewer` if the device cannot give that many; *got says which.  A call that
// finds `fewer` from an earlier shortage moves to `bytes` as soon as the device has them free
// (beside what is held, so that a failed try gives nothing up).
char* hisq_scratch(size_t bytes, size_t fewer, size_t* got)
{
    int dev = 0;
    KS_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_hisq_mu);
    HisqScratch& h = g_hisq[dev];
    auto take = [&](void* p, size_t n) {
        device_free(h.ptr);
        h.ptr = p;
        h.bytes = n;
    };
    if (h.bytes < fewer) take(nullptr, 0);
    size_t room = 0, total = 0;
    if (h.bytes < bytes && (h.bytes == 0 || (hipMemGetInfo(&room, &total) == hipSuccess && room >= bytes))) {
        try {
            take(device_alloc(bytes), bytes);
        } catch (const Failure&) {
            if (h.bytes == 0) take(device_alloc(fewer), fewer);
        }
    }
    *got = h.bytes >= bytes ? bytes : fewer;
    return static_cast<char*>(h.ptr);
}

}  // namespace

void hisq_release()
{
    std::lock_guard<std::mutex> lk(g_hisq_mu);
    int cur = 0;
    (void)hipGetDevice(&cur);
    for (auto& kv : g_hisq) {
        (void)hipSetDevice(kv.first);
        (void)hipDeviceSynchronize();
        device_free(kv.second.ptr);
    }
    (void)hipSetDevice(cur);
    g_hisq.clear();
}

void hisq_links(const Geom& G, const double* thin, double* fat, double* naik,
                const double* level1, const double* level2, double c_naik, hipStream_t st)
{
    const long vol = G.V;
    const size_t field = (size_t)tile_sites(vol) * 9;   // double2 per scratch field
    const size_t fb = field * sizeof(double2);
    const size_t few = 14 * fb + 256, many = 32 * fb + 256;
    size_t got = 0;
    char* base = hisq_scratch(many <= kWideScratch ? many : few, few, &got);
    const int mus = got > few ? 4 : 1;
    double2* U = reinterpret_cast<double2*>(base);
    double2* W = U + 4 * field;
    double2* T = W + 4 * field;
    double2* I = T + 3 * mus * field;
    int* bad = reinterpret_cast<int*>(I + 3 * mus * field);
    const int nb = blocks_for(vol);
    // tile order: needs whole tiles per (z, t) plane
    int pb = 0, zb = 0;
    if (G.n[0] * G.n[1] % kTileSites == 0) {
        pb = divisor_upto(G.n[0] * G.n[1] / kTileSites, 4);
        zb = divisor_upto(G.n[2], 4);
    }
    tile_links_kernel<<<dim3(nb, 4), kBlock, 0, st>>>(G.V, reinterpret_cast<const double2*>(thin), U,
                                                      field);
    KS_HIP(hipGetLastError());
    const SmearArgs a{U,         T,         I,         field, level1[0], level1[1],
                      level1[2], level1[3], level1[4], 0,     pb,        zb};
    if (mus == 4) smear<4, false>(G, a, W, st);
    else smear<1, false>(G, a, W, st);
    KS_HIP(hipMemsetAsync(bad, 0, sizeof(int), st));
    u3_project_kernel<<<dim3(nb, 4), kBlock, 0, st>>>(G.V, W, field, bad);
    KS_HIP(hipGetLastError());
    const SmearArgs b{W,         T,         I,         field, level2[0], level2[1],
                      level2[2], level2[3], level2[4], 0,     pb,        zb};
    double2* fo = reinterpret_cast<double2*>(fat);
    if (mus == 4) smear<4, true>(G, b, fo, st);
    else smear<1, true>(G, b, fo, st);
    naik_kernel<<<dim3(nb, 4), kBlock, 0, st>>>(G, W, field, c_naik, reinterpret_cast<double2*>(naik));
    KS_HIP(hipGetLastError());
    int hbad = 0;
    KS_HIP(hipMemcpyAsync(&hbad, bad, sizeof(int), hipMemcpyDeviceToHost, st));
    KS_HIP(hipStreamSynchronize(st));
    KS_REQUIRE(!hbad, KS_ERR_NONFINITE,
               "link construction: a level-1 smeared link is singular or not finite");
}

}  // namespace ks
