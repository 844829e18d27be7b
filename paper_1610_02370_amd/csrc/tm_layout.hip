// Layout kernels: gauge-link ingest, clover construction, spinor import /
// export between the canonical complex128 layout and the internal tiled
// structure-of-arrays layout, and precision conversion between internal
// fields.
#include "tm_internal.h"

#include <algorithm>

namespace tmsap {

namespace {

constexpr int kThreads = 256;

inline unsigned grid_for(long long n) { return (unsigned)((n + kThreads - 1) / kThreads); }

struct C64 {
    double re, im;
};
__device__ inline C64 cm(C64 a, C64 b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__device__ inline C64 cadd(C64 a, C64 b) { return {a.re + b.re, a.im + b.im}; }
__device__ inline C64 csub(C64 a, C64 b) { return {a.re - b.re, a.im - b.im}; }
__device__ inline C64 cconj(C64 a) { return {a.re, -a.im}; }

struct M3 {
    C64 m[3][3];
};

__device__ inline M3 mmul(const M3& a, const M3& b) {
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            C64 t = cm(a.m[i][0], b.m[0][j]);
            t = cadd(t, cm(a.m[i][1], b.m[1][j]));
            c.m[i][j] = cadd(t, cm(a.m[i][2], b.m[2][j]));
        }
    return c;
}

__device__ inline M3 mdag(const M3& a) {
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) c.m[i][j] = cconj(a.m[j][i]);
    return c;
}

// Coordinates of tiled site s in 32-bit arithmetic (a lattice has at most 2^29 sites).
__device__ inline void coords32(const Geo& g, unsigned s, int c[4]) {
    unsigned blk = s / (unsigned)g.Vb, l = s - blk * (unsigned)g.Vb;
#pragma unroll
    for (int a = 3; a >= 0; --a) {
        const unsigned nb = (unsigned)g.nb[a], lb = (unsigned)g.lb[a], bq = blk / nb, lq = l / lb;
        c[a] = (int)((blk - bq * nb) * lb + (l - lq * lb));
        blk = bq;
        l = lq;
    }
}

// ------------------------------------------------------------ link ingest
// The links of time slices t0 .. t0 + nt (wrapped), 64 sites per workgroup, one (site, direction) per
// thread.  The canonical array is read in its own order through LDS: read link by link, 64 lanes
// touch 64 separate cache lines per load.  Writes, as asked for: the internal two-row copy of the
// slices t0 + k0 .. t0 + k0 + kn (with the SU(3) check), and all nine elements in the staged order `soa`
// [4 mu][nt][z][y][x / 4][9][x % 4]: four neighbouring sites' elements side by side, a link within 640 bytes.
// stats[0]: max deviation from SU(3) (float bits), stats[1]: nonfinite flag.
// 32^3x64 with staging: 0.70 ms for 1.2 GB read and 2.0 GB written (0.51 without the staged copy).
constexpr int kIngestSites = 64;

// Element 0 of the staged link at x of a row (of all directions and slices); element e is at + 4 e.
__device__ inline size_t staged_link(unsigned row, unsigned X, unsigned x) {
    return ((size_t)row * ((X + 3) / 4) + x / 4) * 36 + x % 4;
}

template <class G>
__global__ void __launch_bounds__(kThreads) k_link_ingest(Geo g, const double* __restrict__ U, int t0, int nt, int k0,
                                                          int kn, void* links, unsigned* stats, double2* soa) {
    constexpr int kPitch = 37;  // 36 complex numbers per site, padded: 592 bytes spread over the banks
    __shared__ double2 lds[kIngestSites * kPitch];
    const unsigned S = (unsigned)(g.V / g.d[0]);
    const unsigned per = (S + kIngestSites - 1) / kIngestSites;  // workgroups per slice
    const int k = (int)(blockIdx.x / per);
    const unsigned first = (blockIdx.x - (unsigned)k * per) * kIngestSites;
    const unsigned cnt = min((unsigned)kIngestSites, S - first);
    int t = (t0 + k) % g.d[0];
    const double2* src = reinterpret_cast<const double2*>(U) + ((size_t)t * S + first) * 36;
    for (unsigned i = threadIdx.x; i < cnt * 36; i += kThreads) {
        const unsigned site = i / 36;
        lds[site * kPitch + (i - site * 36)] = src[i];
    }
    __syncthreads();
    const int mu = threadIdx.x >> 6;
    const unsigned n = threadIdx.x & 63;
    const bool on = n < cnt;
    M3 L;
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        const double2 v = on ? lds[n * kPitch + mu * 9 + e] : make_double2(e % 4 == 0 ? 1.0 : 0.0, 0.0);
        L.m[e / 3][e % 3] = {v.x, v.y};
    }
    if (soa && on) {
        const unsigned X = (unsigned)g.d[3], row = (first + n) / X, x = first + n - row * X, rows = S / X;
        double2* o = soa + staged_link((unsigned)(mu * nt + k) * rows + row, X, x);
#pragma unroll
        for (int e = 0; e < 9; ++e) o[4 * e] = make_double2(L.m[e / 3][e % 3].re, L.m[e / 3][e % 3].im);
    }
    if (!links || k < k0 || k >= k0 + kn) return;
    float dev = 0.f;
    bool bad = false;
#pragma unroll
    for (int e = 0; e < 9; ++e) bad |= !isfinite(L.m[e / 3][e % 3].re) || !isfinite(L.m[e / 3][e % 3].im);
    // |U U^+ - 1| and |det U - 1|
    const M3 P = mmul(L, mdag(L));
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const double e = fabs(P.m[i][j].re - (i == j ? 1.0 : 0.0)) + fabs(P.m[i][j].im);
            dev = fmaxf(dev, (float)e);
        }
    C64 det = {0, 0};
    det = cadd(det, cm(L.m[0][0], csub(cm(L.m[1][1], L.m[2][2]), cm(L.m[1][2], L.m[2][1]))));
    det = csub(det, cm(L.m[0][1], csub(cm(L.m[1][0], L.m[2][2]), cm(L.m[1][2], L.m[2][0]))));
    det = cadd(det, cm(L.m[0][2], csub(cm(L.m[1][0], L.m[2][1]), cm(L.m[1][1], L.m[2][0]))));
    dev = fmaxf(dev, (float)(fabs(det.re - 1.0) + fabs(det.im)));
    if (on) {
        const unsigned lex = first + n;
        const int x = (int)(lex % (unsigned)g.d[3]), y = (int)(lex / (unsigned)g.d[3] % (unsigned)g.d[2]),
                  z = (int)(lex / ((unsigned)g.d[3] * (unsigned)g.d[2]));
        const int c[4] = {t, z, y, x};
        const long long s = coords_site(g, c);
        const double u[12] = {L.m[0][0].re, L.m[0][0].im, L.m[0][1].re, L.m[0][1].im, L.m[0][2].re, L.m[0][2].im,
                              L.m[1][0].re, L.m[1][0].im, L.m[1][1].re, L.m[1][1].im, L.m[1][2].re, L.m[1][2].im};
#pragma unroll
        for (int q = 0; q < 3; ++q) Unit<G>::store(links, ((size_t)mu * 3 + q) * g.V + s, u + 4 * q);
    }
    // one atomic per wavefront, and only where there is something to record
    if (!(dev == dev)) dev = 1e30f;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) dev = fmaxf(dev, __shfl_xor(dev, off, 64));
    const bool any_bad = __any(bad);
    if (n == 0) {
        if (any_bad) atomicOr(&stats[1], 1u);
        if (__float_as_uint(dev) > __atomic_load_n(&stats[0], __ATOMIC_RELAXED)) atomicMax(&stats[0], __float_as_uint(dev));
    }
}

// ------------------------------------------------------------ clover build
// A = (m+4) - (c_sw/16) sum_{mu<nu} (gamma_mu gamma_nu) (x) F_munu with F = Q_munu - Q_numu = Q - Q^+, Q the
// four-leaf clover.  In the chiral basis gamma_mu gamma_nu = diag(B_mu B_nu^+, B_mu^+ B_nu) (B_0 = -1,
// B_k = -i sigma_k): the planes (0, l) give -+ i sigma_l and the spatial plane jk with eps_jkl = 1 gives
// i sigma_l in both blocks.  With H_l = i (F_jk -+ F_0l), Hermitian, f = -c_sw/16 and spins as rows:
//   [ m+4 + f H_3        f (H_1 - i H_2) ]
//   [ f (H_1 + i H_2)    m+4 - f H_3     ]
//
// A workgroup holds a box of up to 2 x 4 x 4 x 4 sites (half a 4^4 tile) and goes through the six planes with
// one thread per plaquette: the box's own and those that reach into it from one step below in either direction
// (240 and 200 for 128 sites).  A plaquette's four links give its value around each of its four corners,
// and a corner's anti-Hermitian part, 9 reals, is added to that site's sum in LDS, one corner after the other so
// that every site has one writer.  Two threads per site, one per chirality, then write the blocks.
// 32^3x64: 1.95 ms for the field, 3.2 with one thread per (site, plane) reading the 16 links around its site, 5.55
// with one thread per site.  Two wavefronts per SIMD wait on L2: 1.5 to 1.9 plaquettes of 4 links per site
// and plane; the boxes in XCD order (0.42 GB instead of 0.82 GB from memory per 11 slices) and the staged
// order of the links (one base address and two elements per cache line) are 2.0 of it, from 3.1 ms.

// Where the links come from: the canonical array, or the staged slices tb .. tb + nt.
template <bool STAGED> struct LinkSource {
    static constexpr bool kStaged = STAGED;
    const double2* p;
    int tb, nt;
    __device__ inline M3 get(const Geo& g, const int c[4], int mu) const {
        M3 r;
        if constexpr (STAGED) {
            int k = c[0] - tb;
            if (k < 0) k += g.d[0];
            if (k >= g.d[0]) k -= g.d[0];
            const double2* q = p + staged_link((unsigned)(((mu * nt + k) * g.d[1] + c[1]) * g.d[2] + c[2]),
                                               (unsigned)g.d[3], (unsigned)c[3]);
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                const double2 v = q[4 * e];
                r.m[e / 3][e % 3] = {v.x, v.y};
            }
        } else {
            const double2* q = p + ((size_t)lex_site(g, c) * 4 + mu) * 9;
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                const double2 v = q[e];
                r.m[e / 3][e % 3] = {v.x, v.y};
            }
        }
        return r;
    }
};

__device__ inline void shift(const Geo& g, const int c[4], int a, int dir, int o[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        int v = c[q] + (q == a ? dir : 0);
        if (v < 0) v += g.d[q];
        if (v >= g.d[q]) v -= g.d[q];
        o[q] = v;
    }
}

constexpr int kCloverThreads = 256, kPlanes = 6, kBoxSites = 128;

// The boxes of a build: extents p, boxes per axis, first and last + 1 coordinate.
struct CloverBoxes {
    int p[4], n[4], lo[4], hi[4];
};

// n / e for 0 <= n < 256, 1 <= e <= 8, with inv = ceil(65536 / e)
__device__ inline int small_div(int n, int inv) { return (n * inv) >> 16; }

// Add (or with FIRST, set) -i (Q - Q^+) to the sums of one plane at site n of the box: the diagonal (3 reals)
// and the upper triangle 01, 02, 12 (complex) of the Hermitian matrix.
template <bool FIRST>
__device__ inline void add_corner(const M3& Q, double (*fh)[kBoxSites], int n) {
    double h[9];
#pragma unroll
    for (int i = 0; i < 3; ++i) h[i] = 2.0 * Q.m[i][i].im;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int i = k == 2 ? 1 : 0, j = k == 0 ? 1 : 2;
        const C64 d = csub(Q.m[i][j], cconj(Q.m[j][i]));
        h[3 + 2 * k] = d.im;
        h[4 + 2 * k] = -d.re;
    }
#pragma unroll
    for (int e = 0; e < 9; ++e) fh[e][n] = FIRST ? h[e] : fh[e][n] + h[e];
}

// With a(y) = U_mu(y) U_nu(y+mu) and b(y) = U_nu(y) U_mu(y+nu), the plaquette at y seen from its corners is
// a b^+ at y, U_nu(y+mu) b^+ U_mu(y) at y + mu, b^+ a at y + mu + nu and U_nu(y)^+ a U_mu(y+nu)^+ at y + nu:
// the four leaves of F at those sites.
template <class C, bool STAGED>
__global__ void __launch_bounds__(kCloverThreads) __attribute__((amdgpu_waves_per_eu(2)))
k_clover_build(Geo g, LinkSource<STAGED> src, CloverBoxes bx, double m4, double f, void* clover) {
    __shared__ double fh[kPlanes][9][kBoxSites];
    int org[4];
    {
        int b = (int)xcd_swizzle(blockIdx.x, gridDim.x);
#pragma unroll
        for (int q = 3; q >= 0; --q) {
            org[q] = bx.lo[q] + (b % bx.n[q]) * bx.p[q];
            b /= bx.n[q];
        }
    }
    // site n of the box (x fastest): strides of the box
    const int st[4] = {bx.p[1] * bx.p[2] * bx.p[3], bx.p[2] * bx.p[3], bx.p[3], 1};
#pragma unroll 1
    for (int pl = 0; pl < kPlanes; ++pl) {
        const int mu = pl < 3 ? 0 : (pl < 5 ? 1 : 2), nu = pl < 3 ? pl + 1 : (pl < 5 ? pl - 1 : 3);
        const int am = axis_of(mu), an = axis_of(nu);
        int l[4], y[4], n = threadIdx.x;
        bool on = true;
#pragma unroll
        for (int q = 3; q >= 0; --q) {
            const int e = bx.p[q] + (q == am || q == an ? 1 : 0), m = small_div(n, (65535 + e) / e);
            l[q] = n - m * e - (q == am || q == an ? 1 : 0);
            y[q] = org[q] + l[q];
            on = on && y[q] < bx.hi[q];
            n = m;
        }
        on = on && n == 0;
        int lm = 0, ln = 0, em = 0, en = 0, sm = 0, sn = 0, at = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (!on) y[q] = org[q];  // the spare threads load what others load
            if (y[q] < 0) y[q] += g.d[q];
            if (q == am) lm = l[q], em = min(bx.p[q], bx.hi[q] - org[q]), sm = st[q];
            if (q == an) ln = l[q], en = min(bx.p[q], bx.hi[q] - org[q]), sn = st[q];
            at += l[q] * st[q];
        }
        int ym[4], yn[4];
        shift(g, y, am, +1, ym);
        shift(g, y, an, +1, yn);
        const bool m0 = on && lm >= 0, m1 = on && lm + 1 < em, n0 = ln >= 0, n1 = ln + 1 < en;
        const M3 Un = src.get(g, y, nu), Vm = src.get(g, yn, mu);
        const M3 Um = src.get(g, y, mu), Vn = src.get(g, ym, nu);
        __builtin_amdgcn_sched_barrier(0);
        const M3 b = mmul(Un, Vm);
        M3 a;
        {
            const M3 Q = mmul(Vn, mmul(mdag(b), Um));
            if (m1 && n0) add_corner<true>(Q, fh[pl], at + sm);
            a = mmul(Um, Vn);
        }
        __syncthreads();
        {
            const M3 Q = mmul(a, mdag(b));
            if (m0 && n0) add_corner<false>(Q, fh[pl], at);
        }
        __syncthreads();
        asm volatile("" ::: "memory");  // the last corner reads its two links again instead of keeping 72 registers
        {
            const M3 Q = mmul(mdag(b), a);
            if (m1 && n1) add_corner<false>(Q, fh[pl], at + sm + sn);
        }
        __syncthreads();
        {
            const M3 U2 = src.get(g, y, nu), V2 = src.get(g, yn, mu);
            const M3 Q = mmul(mmul(mdag(U2), a), mdag(V2));
            if (m0 && n1) add_corner<false>(Q, fh[pl], at + sn);
        }
    }
    __syncthreads();
    // the box's sites: 128 threads per chirality
    const int ch = __builtin_amdgcn_readfirstlane(threadIdx.x >> 7);
    const int n = threadIdx.x & (kBoxSites - 1);
    int c[4], r = n;
    bool on = true;
#pragma unroll
    for (int q = 3; q >= 0; --q) {
        const int m = small_div(r, (65535 + bx.p[q]) / bx.p[q]);
        c[q] = org[q] + r - m * bx.p[q];
        on = on && c[q] < bx.hi[q];
        r = m;
    }
    if (!on || r != 0) return;
    const long long s = coords_site(g, c);
    // chirality ch: H_l = i (F_jk -+ F_0l) = -(H_jk -+ H_0l); planes 0..2 are (0, l), 5, 4, 3 the jk of
    // l = 1, 2, 3, plane 4 = (1, 3) with the sign of eps_132
    const double sg = ch == 0 ? -1.0 : 1.0;
    double h[3][9];
#pragma unroll
    for (int l = 0; l < 3; ++l)
#pragma unroll
        for (int e = 0; e < 9; ++e)
            h[l][e] = -f * ((l == 1 ? -1.0 : 1.0) * fh[5 - l][e][n] + sg * fh[l][e][n]);
    // f H_l as a full complex element (i, j)
    auto el = [&](int l, int i, int j) -> C64 {
        if (i == j) return {h[l][i], 0.0};
        const int k = i + j - 1, e = 3 + 2 * k;
        return i < j ? C64{h[l][e], h[l][e + 1]} : C64{h[l][e], -h[l][e + 1]};
    };
    double out[36];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        out[i] = m4 + h[2][i];
        out[3 + i] = m4 - h[2][i];
    }
    int k = 6;
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = i + 1; j < 6; ++j) {
            C64 v;
            if (i < 3 && j >= 3) {  // H_1 - i H_2
                const C64 a = el(0, i, j - 3), b = el(1, i, j - 3);
                v = {a.re + b.im, a.im - b.re};
            } else {
                v = el(2, i % 3, j % 3);
                if (i >= 3) v = {-v.re, -v.im};
            }
            out[k++] = v.re;
            out[k++] = v.im;
        }
#pragma unroll
    for (int u = 0; u < 9; ++u) Unit<C>::store(clover, (size_t)(9 * ch + u) * g.V + s, out + 4 * u);
}

// c_sw = 0: the mass term alone.
template <class C>
__global__ void __launch_bounds__(kThreads) k_clover_mass(long long V, double m4, void* clover) {
    const long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= V) return;
    for (int u = 0; u < 18; ++u) {
        double v[4];
        for (int q = 0; q < 4; ++q) v[q] = (4 * u + q) % 36 < 6 ? m4 : 0.0;
        Unit<C>::store(clover, (size_t)u * V + s, v);
    }
}

// FP32 clover from the FP64 one of the same field: the build rounds its FP64
// result once at the store, so this rounding gives the same values.
__global__ void __launch_bounds__(kThreads) k_clover_to_f32(long long n_units, const double* __restrict__ src,
                                                            float* dst) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_units) return;
    const double4 a = reinterpret_cast<const double4*>(src)[i];
    reinterpret_cast<float4*>(dst)[i] = make_float4((float)a.x, (float)a.y, (float)a.z, (float)a.w);
}

// ------------------------------------------------------------ spinors
// canonical [nsys][V][12] complex128 -> internal
template <class S>
__global__ void __launch_bounds__(kThreads) k_spinor_import(Geo g, int nsys, const double* __restrict__ canon,
                                                            void* data, float* scale, unsigned* flag) {
    long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    int sys = blockIdx.y;
    if (s >= g.V || sys >= nsys) return;
    int c[4];
    site_coords(g, s, c);
    long long lex = lex_site(g, c);
    const double2* p = reinterpret_cast<const double2*>(canon) + ((size_t)sys * g.V + lex) * 12;
    Spinor<double> v;
    bool bad = false;
    for (int i = 0; i < 12; ++i) {
        double2 t = p[i];
        v.v[i] = cmk(t.x, t.y);
        if (!isfinite(t.x) || !isfinite(t.y)) bad = true;
    }
    if (bad) atomicOr(flag, 1u);
    store_spinor<double, S>(reinterpret_cast<char*>(data) + (size_t)sys * 6 * g.V * Unit<S>::bytes,
                            scale ? scale + (size_t)sys * g.V : nullptr, g.V, s, v);
}

template <class S>
__global__ void __launch_bounds__(kThreads) k_spinor_export(Geo g, int nsys, const void* __restrict__ data,
                                                            const float* __restrict__ scale, double* canon) {
    long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    int sys = blockIdx.y;
    if (s >= g.V || sys >= nsys) return;
    int c[4];
    site_coords(g, s, c);
    long long lex = lex_site(g, c);
    Spinor<double> v;
    load_spinor<double, S>(reinterpret_cast<const char*>(data) + (size_t)sys * 6 * g.V * Unit<S>::bytes,
                           scale ? scale + (size_t)sys * g.V : nullptr, g.V, s, v);
    double2* p = reinterpret_cast<double2*>(canon) + ((size_t)sys * g.V + lex) * 12;
    for (int i = 0; i < 12; ++i) p[i] = make_double2(v.v[i].re, v.v[i].im);
}

template <class Si, class So>
__global__ void __launch_bounds__(kThreads) k_spinor_convert(Geo g, int nsys, const void* __restrict__ in,
                                                             const float* __restrict__ in_scale, void* out,
                                                             float* out_scale) {
    long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    int sys = blockIdx.y;
    if (s >= g.V || sys >= nsys) return;
    Spinor<double> v;
    load_spinor<double, Si>(reinterpret_cast<const char*>(in) + (size_t)sys * 6 * g.V * Unit<Si>::bytes,
                            in_scale ? in_scale + (size_t)sys * g.V : nullptr, g.V, s, v);
    store_spinor<double, So>(reinterpret_cast<char*>(out) + (size_t)sys * 6 * g.V * Unit<So>::bytes,
                             out_scale ? out_scale + (size_t)sys * g.V : nullptr, g.V, s, v);
}

}  // namespace

// Even-odd site inverses: thread h takes the site of the requested parity in the pair (2h, 2h+1)
// (one even and one odd site, since the block x-extent is even), forms the
// two chiral blocks A_up + i absmu and A_dn - i absmu of the packed clover
// (A = (m+4) + clover, Hermitian) and inverts each by Gauss-Jordan with
// partial pivoting in FP64.
template <class C>
__global__ void __launch_bounds__(kThreads) k_eo_inverse(Geo g, const void* __restrict__ clover, double absmu,
                                                         int parity, void* inv) {
    const long long h = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long half = g.V / 2;
    if (h >= half) return;
    long long s = 2 * h;
    int c[4];
    site_coords(g, s, c);
    if (((c[0] + c[1] + c[2] + c[3]) & 1) != parity) ++s;
    Clover<double> A;
    load_clover<double, C>(clover, g.V, s, A);
    for (int blk = 0; blk < 2; ++blk) {
        const double* P = A.a + 36 * blk;
        const double tw = blk == 0 ? absmu : -absmu;
        cplx<double> M[6][6], X[6][6];
        for (int i = 0; i < 6; ++i)
            for (int j = 0; j < 6; ++j) {
                M[i][j] = cmk(0.0, 0.0);
                X[i][j] = cmk(i == j ? 1.0 : 0.0, 0.0);
            }
        for (int i = 0; i < 6; ++i) M[i][i] = cmk(P[i], tw);
        int k = 6;
        for (int i = 0; i < 6; ++i)
            for (int j = i + 1; j < 6; ++j) {
                M[i][j] = cmk(P[k], P[k + 1]);
                M[j][i] = cmk(P[k], -P[k + 1]);
                k += 2;
            }
        for (int col = 0; col < 6; ++col) {
            int p = col;
            double best = M[col][col].re * M[col][col].re + M[col][col].im * M[col][col].im;
            for (int i = col + 1; i < 6; ++i) {
                const double m2 = M[i][col].re * M[i][col].re + M[i][col].im * M[i][col].im;
                if (m2 > best) {
                    best = m2;
                    p = i;
                }
            }
            if (p != col)
                for (int j = 0; j < 6; ++j) {
                    cplx<double> t = M[col][j];
                    M[col][j] = M[p][j];
                    M[p][j] = t;
                    t = X[col][j];
                    X[col][j] = X[p][j];
                    X[p][j] = t;
                }
            const cplx<double> d = M[col][col];
            const double dn = 1.0 / (d.re * d.re + d.im * d.im);
            const cplx<double> di = cmk(d.re * dn, -d.im * dn);
            for (int j = 0; j < 6; ++j) {
                M[col][j] = di * M[col][j];
                X[col][j] = di * X[col][j];
            }
            for (int i = 0; i < 6; ++i) {
                if (i == col) continue;
                const cplx<double> f = M[i][col];
                for (int j = 0; j < 6; ++j) {
                    M[i][j] = M[i][j] - f * M[col][j];
                    X[i][j] = X[i][j] - f * X[col][j];
                }
            }
        }
        for (int u = 0; u < 18; ++u) {
            const int e0 = 2 * u, e1 = 2 * u + 1;
            const double w[4] = {X[e0 / 6][e0 % 6].re, X[e0 / 6][e0 % 6].im, X[e1 / 6][e1 % 6].re,
                                 X[e1 / 6][e1 % 6].im};
            Unit<C>::store(inv, (size_t)(18 * blk + u) * half + h, w);
        }
    }
}

#define TM_DISPATCH_PREC(P, T, ...)                  \
    switch (P) {                                     \
        case P_F64: { typedef double T; __VA_ARGS__; break; } \
        case P_F32: { typedef float T; __VA_ARGS__; break; }  \
        case P_F16: { typedef f16 T; __VA_ARGS__; break; }    \
        default: { typedef bf16 T; __VA_ARGS__; break; }      \
    }

size_t gauge_stage_bytes(const Geo& g, int slices) {
    return (size_t)slices * (size_t)(g.d[1] * g.d[2]) * (size_t)((g.d[3] + 3) / 4 * 4) * 36 * sizeof(double2);
}

hipError_t launch_link_ingest(const Geo& g, Prec G, const void* Ucanon, void* links, unsigned* stats,
                              hipStream_t st) {
    const unsigned per = grid_for(g.V / g.d[0] * (kThreads / kIngestSites));
    TM_DISPATCH_PREC(G, T, hipLaunchKernelGGL(k_link_ingest<T>, dim3(per * (unsigned)g.d[0]), dim3(kThreads), 0, st, g,
                                              (const double*)Ucanon, 0, g.d[0], 0, g.d[0], links, stats,
                                              (double2*)nullptr));
    return hipGetLastError();
}

hipError_t launch_gauge_build(const Geo& g, Prec G, Prec C, const void* Ucanon, double m4, double csw, void* links,
                              void* clover, unsigned* stats, void* stage, size_t stage_bytes, hipStream_t st) {
    if (C == P_F16 || C == P_BF16) return hipErrorInvalidValue;
    hipError_t e;
    const double f = -csw / 16.0;
    if (csw == 0.0) {
        if ((e = launch_link_ingest(g, G, Ucanon, links, stats, st)) != hipSuccess) return e;
        TM_DISPATCH_PREC(C, T, hipLaunchKernelGGL(k_clover_mass<T>, dim3(grid_for(g.V)), dim3(kThreads), 0, st, g.V, m4,
                                                  clover));
        return hipGetLastError();
    }
    const long long S = g.V / g.d[0];
    const int T = g.d[0], lt = g.lb[0];
    const size_t slice = gauge_stage_bytes(g, 1);
    const int room = (int)(stage ? stage_bytes / slice : 0);
    CloverBoxes bx;
    for (int q = 0; q < 4; ++q) {  // an axis in steps of 4, or of 3 where that pads less (2 and 1 in t)
        const int big = q == 0 ? 2 : 4, small = q == 0 ? 1 : 3, d = g.d[q];
        bx.p[q] = std::min(d, (d + big - 1) / big * big <= (d + small - 1) / small * small ? big : small);
        bx.n[q] = (d + bx.p[q] - 1) / bx.p[q];
        bx.lo[q] = 0;
        bx.hi[q] = d;
    }
    auto build = [&](auto src, int t0, int nt) {  // slices t0 .. t0 + nt
        bx.lo[0] = t0;
        bx.hi[0] = t0 + nt;
        bx.n[0] = (nt + bx.p[0] - 1) / bx.p[0];
        const unsigned nwg = (unsigned)((long long)bx.n[0] * bx.n[1] * bx.n[2] * bx.n[3]);
        TM_DISPATCH_PREC(C, Tc, hipLaunchKernelGGL((k_clover_build<Tc, decltype(src)::kStaged>), dim3(nwg),
                                                   dim3(kCloverThreads), 0, st, g, src, bx, m4, f, clover));
    };
    if (room < T && room < lt + 2) {  // no room to stage one row of tiles with its neighbours
        if ((e = launch_link_ingest(g, G, Ucanon, links, stats, st)) != hipSuccess) return e;
        build(LinkSource<false>{(const double2*)Ucanon, 0, 0}, 0, T);
        return hipGetLastError();
    }
    // whole rows of tiles (contiguous in the tiled layout) with one slice on either side, or everything at once
    const int n = room >= T ? T : (room - 2) / lt * lt;
    const unsigned per = grid_for(S * (kThreads / kIngestSites));
    for (int t = 0; t < T; t += n) {
        const int m = n < T - t ? n : T - t;
        const bool all = n == T;
        const int tb = all ? 0 : (t + T - 1) % T, nt = all ? T : m + 2, k0 = all ? 0 : 1;
        TM_DISPATCH_PREC(G, Tg, hipLaunchKernelGGL(k_link_ingest<Tg>, dim3(per * (unsigned)nt), dim3(kThreads), 0, st, g,
                                                   (const double*)Ucanon, tb, nt, k0, m, links, stats,
                                                   (double2*)stage));
        if ((e = hipGetLastError()) != hipSuccess) return e;
        build(LinkSource<true>{(const double2*)stage, tb, nt}, t, m);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_clover_to_f32(const Geo& g, const void* clover64, void* clover32, hipStream_t st) {
    const long long n = 18 * g.V;
    hipLaunchKernelGGL(k_clover_to_f32, dim3(grid_for(n)), dim3(kThreads), 0, st, n,
                       static_cast<const double*>(clover64), static_cast<float*>(clover32));
    return hipGetLastError();
}

hipError_t launch_spinor_import(const Geo& g, const SpinorBuf& dst, const void* canon, unsigned* flag,
                                hipStream_t st) {
    dim3 grid(grid_for(g.V), dst.nsys);
    TM_DISPATCH_PREC(dst.prec, T, hipLaunchKernelGGL(k_spinor_import<T>, grid, dim3(kThreads), 0, st, g, dst.nsys,
                                                     (const double*)canon, dst.data, dst.scale, flag));
    return hipGetLastError();
}

hipError_t launch_spinor_export(const Geo& g, const SpinorBuf& src, void* canon, hipStream_t st) {
    dim3 grid(grid_for(g.V), src.nsys);
    TM_DISPATCH_PREC(src.prec, T, hipLaunchKernelGGL(k_spinor_export<T>, grid, dim3(kThreads), 0, st, g, src.nsys,
                                                     src.data, src.scale, (double*)canon));
    return hipGetLastError();
}

hipError_t launch_spinor_convert(const Geo& g, const SpinorBuf& src, const SpinorBuf& dst, hipStream_t st) {
    dim3 grid(grid_for(g.V), src.nsys);
    TM_DISPATCH_PREC(src.prec, Ti,
                     TM_DISPATCH_PREC(dst.prec, To,
                                      hipLaunchKernelGGL((k_spinor_convert<Ti, To>), grid, dim3(kThreads), 0, st, g,
                                                         src.nsys, src.data, src.scale, dst.data, dst.scale)));
    return hipGetLastError();
}

hipError_t launch_eo_inverse(const Geo& g, Prec C, const void* clover, double absmu, int parity, void* inv,
                             hipStream_t st) {
    if (C != P_F64 && C != P_F32) return hipErrorInvalidValue;
    const long long half = g.V / 2;
    const unsigned nb = (unsigned)((half + kThreads - 1) / kThreads);
    TM_DISPATCH_PREC(C, T, hipLaunchKernelGGL(k_eo_inverse<T>, dim3(nb > 0 ? nb : 1), dim3(kThreads), 0, st, g,
                                              clover, absmu, parity, inv));
    return hipGetLastError();
}

}  // namespace tmsap
