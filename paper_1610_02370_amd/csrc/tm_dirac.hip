// The twisted-mass Wilson-clover operator on the whole lattice
// (section 2.1): out = [(m+4) + C + i mu Gamma5] psi
//   - 1/2 sum_mu [(1 - gamma_mu) U_mu(x) psi(x+mu) + (1 + gamma_mu) U_mu(x-mu)^+ psi(x-mu)].
// One thread per site; spin projection to half spinors before the SU(3)
// products; every field is read structure-of-arrays so a wavefront's loads
// are contiguous.
#include <type_traits>

#include "tm_internal.h"
#include "tm_pair.h"

namespace tmsap {

namespace {

constexpr int kThreads = 256;
// Up to here (sites times systems) the FP64 operator splits the directions over wavefronts: below, one
// workgroup of the unsplit kernel or less falls on each compute unit.  All FP64 kernels form the same products and
// add them in the same order: a system's result is the same bits whatever the number of systems selects.
constexpr long long kSplitSites = 32768;

// Link from its first two rows, stored as 12 reals (row-major, re/im pairs); third row rebuilt.
template <class R>
__device__ inline void link_from_rows(const R* u, Link<R>& L) {
    L.u[0][0] = cmk(u[0], u[1]);
    L.u[0][1] = cmk(u[2], u[3]);
    L.u[0][2] = cmk(u[4], u[5]);
    L.u[1][0] = cmk(u[6], u[7]);
    L.u[1][1] = cmk(u[8], u[9]);
    L.u[1][2] = cmk(u[10], u[11]);
    complete_su3(L);
}

template <class Si, class So, class G, class C, class R>
__global__ void __launch_bounds__(kThreads) k_dirac(DiracArgs a) {
    const Geo& g = a.g;
    // workgroups of one XCD on consecutive tiles (their neighbours' spinors and links share an L2)
    long long s = xcd_swizzle(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (s >= g.V) return;
    int nf[4], nbk[4], par;
    unsigned wrap;
    tiled_neighbours(g, s, nf, nbk, &wrap, &par);
    Clover<R> A;
    load_clover<R, C>(a.clover, g.V, s, A);
    // FP32 spinors and links: the 8 links of the site's hops (two rows each) are loaded once
    // for all systems.  The FP16 / BF16 forms reload them per system: holding them takes these
    // kernels to one wavefront per SIMD, which costs more than the loads.
    constexpr bool kHold = std::is_same<Si, float>::value && std::is_same<G, float>::value &&
                           std::is_same<R, float>::value;
    R lr[kHold ? 8 : 1][12];
    if constexpr (kHold) {
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) {
            const size_t b = (size_t)mu * 3 * g.V;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                Unit<G>::load(a.links, b + (size_t)q * g.V + s, &lr[2 * mu][4 * q]);
                Unit<G>::load(a.links, b + (size_t)q * g.V + nbk[mu], &lr[2 * mu + 1][4 * q]);
            }
        }
    }
    const size_t in_stride = (size_t)6 * g.V * Unit<Si>::bytes;
    const size_t out_stride = (size_t)6 * g.V * Unit<So>::bytes;
    const int sys_begin = blockIdx.y * a.sys_tile;
    const int sys_end = min(a.nsys, sys_begin + a.sys_tile);
    for (int sys = sys_begin; sys < sys_end; ++sys) {
        const void* in = reinterpret_cast<const char*>(a.in) + sys * in_stride;
        const float* isc = a.in_scale ? a.in_scale + (size_t)sys * g.V : nullptr;
        Spinor<R> acc;
#pragma unroll
        for (int i = 0; i < 12; ++i) acc.v[i] = cmk<R>(0, 0);
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) {
            Link<R> L;
            Spinor<R> p;
            if constexpr (kHold)
                link_from_rows(lr[2 * mu], L);
            else
                load_link<R, G>(a.links, g.V, s, mu, L);
            load_spinor<R, Si>(in, isc, g.V, nf[mu], p);
            {  // boundary phase (1 for hops inside the lattice), branch-free: fewer registers
                const bool w = wrap & (1u << mu);
                const R re = w ? (R)g.bcr[mu] : (R)1, im = w ? (R)g.bci[mu] : (R)0;
#pragma unroll
                for (int i = 0; i < 12; ++i) p.v[i] = cmk(re * p.v[i].re - im * p.v[i].im, re * p.v[i].im + im * p.v[i].re);
            }
            hop_forward(mu, L, p, (R)1, acc);
            if constexpr (kHold)
                link_from_rows(lr[2 * mu + 1], L);
            else
                load_link<R, G>(a.links, g.V, nbk[mu], mu, L);
            load_spinor<R, Si>(in, isc, g.V, nbk[mu], p);
            {
                const bool w = wrap & (16u << mu);
                const R re = w ? (R)g.bcr[mu] : (R)1, im = w ? -(R)g.bci[mu] : (R)0;
#pragma unroll
                for (int i = 0; i < 12; ++i) p.v[i] = cmk(re * p.v[i].re - im * p.v[i].im, re * p.v[i].im + im * p.v[i].re);
            }
            hop_backward(mu, L, p, (R)1, acc);
        }
        Spinor<R> self, out;
        load_spinor<R, Si>(in, isc, g.V, s, self);
        clover_apply(A, (R)(a.mu[sys] + g.mu_shift[par]), self, out);
#pragma unroll
        for (int i = 0; i < 12; ++i) out.v[i] = out.v[i] - (R)0.5 * acc.v[i];
        store_spinor<R, So>(reinterpret_cast<char*>(a.out) + sys * out_stride,
                            a.out_scale ? a.out_scale + (size_t)sys * g.V : nullptr, g.V, s, out);
    }
}

// FP64, one lane per site, in the internal layout, mostly for several systems.  STAGED (4^4 tiles, one per workgroup): the
// workgroup stages its tile's own links (two rows each, 96 KiB) in LDS once, and every system takes its
// forward links there; on other tiles they too come from memory per system.  The backward links U_mu(x - mu) stay loads from memory: inside the tile they are the
// links just staged, still in L2, and read from LDS as well they made the compiler spill a kilobyte per lane.
// 32^3x64 in 820 us for one system and 465 per system for six, against 800 and 700 with two lanes per site
// (k_dirac_pair), whose neighbour reads all go to L2.  Products and sums are those of the pair's two lanes, in
// their order; the phase after the projection, on 6 numbers instead of 12, took 2 to 5 % off.
template <int MU, int DIR>
__device__ inline void site_hop(const Geo& g, const Spinor<double>& psi, const cplx<double> u[6], bool wrap,
                                PairAcc<double> acc[2]) {
    // boundary phase (1 for hops inside the lattice), branch-free: fewer registers
    const cplx<double> ph = cmk(wrap ? g.bcr[MU] : 1.0, wrap ? (DIR > 0 ? g.bci[MU] : -g.bci[MU]) : 0.0);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const double s = c != 0 ? 1.0 : -1.0;
        Col<double> p, q, h, t;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            p.v[k] = psi.v[3 * c + k];
            q.v[k] = psi.v[3 * (pair_cross(MU) ? 3 - c : 2 + c) + k];
        }
        pair_project<MU, DIR>(p, q, s, h);
#pragma unroll
        for (int k = 0; k < 3; ++k) h.v[k] = mul_fixed(ph, h.v[k]);
        if constexpr (DIR > 0)
            pair_mul_fixed(u, h, t);
        else
            pair_dag_mul_fixed(u, h, t);
        pair_accumulate<MU, DIR>(t, s, acc[c]);
    }
}

// Both hops of direction MU into the site; `fwd` its own link.
template <int MU>
__device__ inline void site_dir(const DiracArgs& a, const void* in, const cplx<double> fwd[6], const int nf[4],
                                const int nbk[4], unsigned wrap, PairAcc<double> acc[2]) {
    Spinor<double> p;
    load_spinor<double, double>(in, nullptr, a.g.V, nf[MU], p);
    site_hop<MU, +1>(a.g, p, fwd, wrap & (1u << MU), acc);
    cplx<double> u[6];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        double w[4];
        Unit<double>::load(a.links, (size_t)(3 * MU + q) * a.g.V + nbk[MU], w);
        u[2 * q] = cmk(w[0], w[1]);
        u[2 * q + 1] = cmk(w[2], w[3]);
    }
    load_spinor<double, double>(in, nullptr, a.g.V, nbk[MU], p);
    site_hop<MU, -1>(a.g, p, u, wrap & (16u << MU), acc);
}

template <bool STAGED>
__global__ void __launch_bounds__(kThreads) k_dirac_lk(DiracArgs a) {
    __shared__ double2 lk[STAGED ? 4 : 1][6][STAGED ? kThreads : 1];  // [mu][row-major pair][site in tile]
    const Geo& g = a.g;
    const long long tile = xcd_swizzle(blockIdx.x, gridDim.x);
    const int l = threadIdx.x;
    const long long s = tile * kThreads + l;  // staged: V is a multiple of the tile size
    const double2* src = reinterpret_cast<const double2*>(a.links);
    if constexpr (STAGED) {
#pragma unroll
        for (int mu = 0; mu < 4; ++mu)
#pragma unroll
            for (int q = 0; q < 3; ++q) {  // unit q of a link holds 4 reals: pairs 2q and 2q+1
                const size_t u = ((size_t)mu * 3 + q) * g.V + s;
                lk[mu][2 * q][l] = src[2 * u];
                lk[mu][2 * q + 1][l] = src[2 * u + 1];
            }
    } else if (s >= g.V) {
        return;
    }
    int nf[4], nbk[4], par;
    unsigned wrap;
    tiled_neighbours(g, s, nf, nbk, &wrap, &par);
    Clover<double> A;
    load_clover<double, double>(a.clover, g.V, s, A);
    if constexpr (STAGED) __syncthreads();
    const size_t stride = (size_t)6 * g.V * Unit<double>::bytes;
    const int sys_begin = blockIdx.y * a.sys_tile;
    const int sys_end = min(a.nsys, sys_begin + a.sys_tile);
    for (int sys = sys_begin; sys < sys_end; ++sys) {
        const void* in = reinterpret_cast<const char*>(a.in) + sys * stride;
        // the thread index again through a barrier the compiler cannot see through: the reads of the
        // links do not depend on the system, and hoisted out of this loop they would be held in
        // registers
        const int lx = opaque(l);
        const auto own = [&](int mu, cplx<double> u[6]) {
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                double2 v;
                if constexpr (STAGED)
                    v = lk[mu][k][lx];
                else
                    v = src[2 * (((size_t)mu * 3 + k / 2) * g.V + tile * kThreads + lx) + k % 2];
                u[k] = cmk(v.x, v.y);
            }
        };
        PairAcc<double> acc[2];
        pair_zero(acc[0]);
        pair_zero(acc[1]);
        cplx<double> u[6];
        own(0, u);
        site_dir<0>(a, in, u, nf, nbk, wrap, acc);
        own(1, u);
        site_dir<1>(a, in, u, nf, nbk, wrap, acc);
        own(2, u);
        site_dir<2>(a, in, u, nf, nbk, wrap, acc);
        own(3, u);
        site_dir<3>(a, in, u, nf, nbk, wrap, acc);
        Spinor<double> self, hop, out;
#pragma unroll
        for (int k = 0; k < 3; ++k) {  // as pair_finish
            hop.v[k] = acc[0].up.v[k];
            hop.v[3 + k] = acc[1].up.v[k];
            hop.v[6 + k] = acc[0].same.v[k] + acc[1].cross.v[k];
            hop.v[9 + k] = acc[0].cross.v[k] + acc[1].same.v[k];
        }
        load_spinor<double, double>(in, nullptr, g.V, s, self);
        clover_apply(A, a.mu[sys] + g.mu_shift[par], self, out);
#pragma unroll
        for (int i = 0; i < 12; ++i) out.v[i] = out.v[i] - 0.5 * hop.v[i];
        store_spinor<double, double>(reinterpret_cast<char*>(a.out) + sys * stride, nullptr, g.V, s, out);
    }
}

// ---------------------------------------------------------------------------
// FP64 arithmetic: two lanes per site (tm_pair.h), any tiles, fields in the internal layout (any
// storage in) or in the canonical one, which spares the conversions of canonical buffers.
//
// At FP64 one lane per site holds the clover and little else at one wavefront per SIMD, and waits for its
// neighbours one hop at a time.  A pair's lanes each read the two spins of a neighbour that their
// half spinor needs, and both hops of a direction are read before either is used.
//
// Measured, with the calls' canonical buffers: 6x10x7x9, 3 systems, 26.6 -> 13.3 us a call; 4^4, 2 systems, 19.6
// -> 13.2 (7.9 and 6.0 us of it the kernel); 32^3x64, one, two and twelve systems 1150 -> 790, 1914 -> 1335 and
// 9900 -> 6970.  FP32 in and FP64 out (any number of systems: the halved reads leave nothing to the one-lane
// kernel), 32^3x64, 2 / 3 / 6 / 12 systems 1736 / 2471 / 4872 / 9810 -> 1068 / 1509 / 2885 / 5515; 24^4 in 4^3x2 tiles, 12
// systems 1666 -> 817, BF16 in 1288 -> 725.  Large lattices are bound by the neighbours' reads from L2 (about 3 KB
// per site and system, 8 to 9 TB/s).

// The canonical layout as a field (FieldOf, tm_pair.h, is the internal one).
struct Canonical {
    const double2* base;
    __device__ inline Canonical(const void* p, const float*, int sys, const Geo& g)
        : base(static_cast<const double2*>(p) + (size_t)sys * 12 * g.V) {}
    __device__ inline void chirality(long long lex, int c, Chir<double>& v) const {
        const double2* r = base + 12 * (size_t)lex + 6 * c;
#pragma unroll
        for (int i = 0; i < 6; ++i) v.v[i] = cmk(r[i].x, r[i].y);
    }
    struct Raw {
        Col<double> p, q;
    };
    template <int MU> __device__ inline void read(long long lex, int c, Raw& r) const {
        const double2* a = base + 12 * (size_t)lex + 3 * c;
        const double2* b = base + 12 * (size_t)lex + 3 * (pair_cross(MU) ? 3 - c : 2 + c);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            r.p.v[k] = cmk(a[k].x, a[k].y);
            r.q.v[k] = cmk(b[k].x, b[k].y);
        }
    }
    template <int MU> static __device__ inline void spins(const Raw& r, int, Col<double>& p, Col<double>& q) {
        p = r.p;
        q = r.q;
    }
    static constexpr bool kCanonical = true;
};

// The product that one hop adds (pair_accumulate).
template <int MU, int DIR, class F>
__device__ inline void hop_term(const Geo& g, const typename F::Raw& psi, const cplx<double> u[6], bool wrap, int c,
                                double s, Col<double>& t) {
    Col<double> p, q, h;
    F::template spins<MU>(psi, c, p, q);
    pair_project<MU, DIR>(p, q, s, h);
    if (wrap) {  // boundary phase
        const cplx<double> ph = cmk(g.bcr[MU], DIR > 0 ? g.bci[MU] : -g.bci[MU]);
#pragma unroll
        for (int k = 0; k < 3; ++k) h.v[k] = mul_fixed(ph, h.v[k]);
    }
    if constexpr (DIR > 0)
        pair_mul_fixed(u, h, t);
    else
        pair_dag_mul_fixed(u, h, t);
}

// The site's neighbours: tiled (links) and, for canonical fields, lexicographic.
struct PairSite {
    long long s, lex;
    int nf[4], nbk[4], cf[4], cb[4];
    unsigned wrap;
    int parity;
};
template <bool CANON> __device__ inline void pair_site(const Geo& g, long long s, PairSite& t) {
    t.s = s;
    tiled_neighbours(g, s, t.nf, t.nbk, &t.wrap, &t.parity);
    t.lex = s;
    if constexpr (CANON) {
        unsigned blk = (unsigned)s / (unsigned)g.Vb, l = (unsigned)s - blk * (unsigned)g.Vb;
        int c[4], st[4];
#pragma unroll
        for (int a = 3; a >= 0; --a) {
            const unsigned nb = (unsigned)g.nb[a], lb = (unsigned)g.lb[a], bq = blk / nb, lq = l / lb;
            c[a] = (int)((blk - bq * nb) * lb + (l - lq * lb));
            blk = bq;
            l = lq;
        }
        st[3] = 1;
#pragma unroll
        for (int a = 2; a >= 0; --a) st[a] = st[a + 1] * g.d[a + 1];
        const int lex = c[0] * st[0] + c[1] * st[1] + c[2] * st[2] + c[3];
        t.lex = lex;
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) {
            const int a = axis_of(mu), span = (g.d[a] - 1) * st[a];
            t.cf[mu] = c[a] + 1 < g.d[a] ? lex + st[a] : lex - span;
            t.cb[mu] = c[a] > 0 ? lex - st[a] : lex + span;
        }
    }
}

// What both hops of direction MU need from memory.
template <class F> struct DirOperands {
    cplx<double> uf[6], ub[6];
    typename F::Raw pf, pb;
};
template <int MU, class F>
__device__ inline void dir_read(const DiracArgs& a, const F& in, const PairSite& t, int c, DirOperands<F>& d) {
    in.template read<MU>(F::kCanonical ? t.cf[MU] : t.nf[MU], c, d.pf);
    link_read<MU>(a.links, a.g.V, t.s, c, d.uf);
    in.template read<MU>(F::kCanonical ? t.cb[MU] : t.nbk[MU], c, d.pb);
    link_read<MU>(a.links, a.g.V, t.nbk[MU], c, d.ub);
}

// Both hops of direction MU.
template <int MU, class F>
__device__ inline void dir_add(const DiracArgs& a, const F& in, const PairSite& t, int c, double s,
                               PairAcc<double>& acc) {
    __builtin_amdgcn_sched_barrier(0);  // one direction's operands live at a time
    DirOperands<F> d;
    dir_read<MU>(a, in, t, c, d);
    Col<double> v;
    hop_term<MU, +1, F>(a.g, d.pf, d.uf, t.wrap & (1u << MU), c, s, v);
    pair_accumulate<MU, +1>(v, s, acc);
    hop_term<MU, -1, F>(a.g, d.pb, d.ub, t.wrap & (16u << MU), c, s, v);
    pair_accumulate<MU, -1>(v, s, acc);
    pin(acc);
    __builtin_amdgcn_sched_barrier(0);
}

// Clover, twist and the store for one system, its hop sum formed.
template <class F, class So>
__device__ inline void site_finish(const DiracArgs& a, int sys, const PairSite& t, int c, const double A[36], bool on,
                                   const PairAcc<double>& acc) {
    const Geo& g = a.g;
    const bool lower = c != 0;
    const F in(a.in, a.in_scale, sys, g);
    Chir<double> hop, self, out;
    pair_finish(acc, lower, hop);
    in.chirality(t.lex, c, self);
    const double mu = a.mu[sys] + g.mu_shift[t.parity];
    clover_block_apply(A, lower ? -mu : mu, self.v, out.v);
#pragma unroll
    for (int i = 0; i < 6; ++i) out.v[i] = out.v[i] - 0.5 * hop.v[i];
    if (!on) return;
    if constexpr (F::kCanonical) {
        double2* o = static_cast<double2*>(a.out) + ((size_t)sys * g.V + t.lex) * 12 + 6 * c;
#pragma unroll
        for (int i = 0; i < 6; ++i) o[i] = make_double2(out.v[i].re, out.v[i].im);
    } else {
        store_chir<double, So>(static_cast<char*>(a.out) + (size_t)sys * 6 * g.V * Unit<So>::bytes, nullptr, g.V, t.s, c,
                               out);
    }
}

__device__ inline void clover_read(const DiracArgs& a, size_t s, int c, double A[36]) {
    const size_t at = (size_t)(9 * c) * a.g.V + s;
#pragma unroll
    for (int k = 0; k < 9; ++k) Unit<double>::load(plane<double>(a.clover, k, a.g.V), at, A + 4 * k);
}

// 32 sites of one system per wavefront.  The four wavefronts of a workgroup take `sys_tile` (1, 2 or 4)
// systems of the same sites, so that the later ones find the links and the clover in the vector cache.
template <class F, class So>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) k_dirac_pair(DiracArgs a) {
    const Geo& g = a.g;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, c = lane & 1;
    const double s = c != 0 ? 1.0 : -1.0;
    const int groups = 4 / a.sys_tile, sys = blockIdx.y * a.sys_tile + w / groups;
    if (sys >= a.nsys) return;
    // workgroups of one XCD on consecutive sites (their neighbours' spinors and links share an L2)
    const long long at = (xcd_swizzle(blockIdx.x, gridDim.x) * groups + w % groups) * 32 + (lane >> 1);
    const bool on = at < g.V;
    PairSite t;
    pair_site<F::kCanonical>(g, on ? at : 0, t);
    const F in(a.in, a.in_scale, sys, g);
    PairAcc<double> acc;
    pair_zero(acc);
    dir_add<0>(a, in, t, c, s, acc);
    dir_add<1>(a, in, t, c, s, acc);
    dir_add<2>(a, in, t, c, s, acc);
    dir_add<3>(a, in, t, c, s, acc);
    double A[36];
    clover_read(a, (size_t)t.s, c, A);
    site_finish<F, So>(a, sys, t, c, A, on, acc);
}

// 32 sites of one system per workgroup, wavefront w on direction w; the products meet in LDS, and the first
// wavefront adds them up in k_dirac_pair's order.
template <int MU, class F>
__device__ inline void dir_terms(const DiracArgs& a, const F& in, const PairSite& t, int c, double s, Col<double>& f,
                                 Col<double>& b) {
    DirOperands<F> d;
    dir_read<MU>(a, in, t, c, d);
    hop_term<MU, +1, F>(a.g, d.pf, d.uf, t.wrap & (1u << MU), c, s, f);
    hop_term<MU, -1, F>(a.g, d.pb, d.ub, t.wrap & (16u << MU), c, s, b);
}
template <int MU>
__device__ inline void dir_sum(const double2 (&part)[3][6][64], int lane, double s, PairAcc<double>& acc) {
    Col<double> v;
#pragma unroll
    for (int k = 0; k < 3; ++k) v.v[k] = cmk(part[MU - 1][k][lane].x, part[MU - 1][k][lane].y);
    pair_accumulate<MU, +1>(v, s, acc);
#pragma unroll
    for (int k = 0; k < 3; ++k) v.v[k] = cmk(part[MU - 1][3 + k][lane].x, part[MU - 1][3 + k][lane].y);
    pair_accumulate<MU, -1>(v, s, acc);
}

template <class F, class So>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) k_dirac_pair_split(DiracArgs a) {
    __shared__ double2 part[3][6][64];
    const Geo& g = a.g;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, c = lane & 1;
    const double s = c != 0 ? 1.0 : -1.0;
    const long long at = (long long)blockIdx.x * 32 + (lane >> 1);
    const bool on = at < g.V;
    const int sys = blockIdx.y;
    PairSite t;
    pair_site<F::kCanonical>(g, on ? at : 0, t);
    double A[36];
    if (w == 0) clover_read(a, (size_t)t.s, c, A);
    const F in(a.in, a.in_scale, sys, g);
    Col<double> f, b;
    switch (w) {
        case 0: dir_terms<0>(a, in, t, c, s, f, b); break;
        case 1: dir_terms<1>(a, in, t, c, s, f, b); break;
        case 2: dir_terms<2>(a, in, t, c, s, f, b); break;
        default: dir_terms<3>(a, in, t, c, s, f, b); break;
    }
    if (w > 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            part[w - 1][k][lane] = make_double2(f.v[k].re, f.v[k].im);
            part[w - 1][3 + k][lane] = make_double2(b.v[k].re, b.v[k].im);
        }
    }
    __syncthreads();
    if (w > 0) return;
    PairAcc<double> acc;
    pair_zero(acc);
    pair_accumulate<0, +1>(f, s, acc);
    pair_accumulate<0, -1>(b, s, acc);
    dir_sum<1>(part, lane, s, acc);
    dir_sum<2>(part, lane, s, acc);
    dir_sum<3>(part, lane, s, acc);
    site_finish<F, So>(a, sys, t, c, A, on, acc);
}

template <class F, class So>
hipError_t run_pair(const DiracArgs& args, hipStream_t st) {
    DiracArgs a = args;
    if (a.g.V * a.nsys <= kSplitSites) {
        hipLaunchKernelGGL((k_dirac_pair_split<F, So>), dim3((unsigned)((a.g.V + 31) / 32), (unsigned)a.nsys),
                           dim3(kThreads), 0, st, a);
    } else {
        a.sys_tile = a.nsys > 2 ? 4 : a.nsys;
        const long long per = 128 / a.sys_tile;  // sites of a workgroup
        hipLaunchKernelGGL((k_dirac_pair<F, So>), dim3((unsigned)((a.g.V + per - 1) / per),
                           (unsigned)((a.nsys + a.sys_tile - 1) / a.sys_tile)), dim3(kThreads), 0, st, a);
    }
    return hipGetLastError();
}

template <class Si, class So, class G, class C, class R>
hipError_t run(const DiracArgs& args, hipStream_t st) {
    DiracArgs a = args;
    const unsigned nwg = (unsigned)((a.g.V + kThreads - 1) / kThreads);
    a.sys_tile = pick_sys_tile(nwg, a.nsys, kCUs, 0.4, true);
    const dim3 grid(nwg, (unsigned)((a.nsys + a.sys_tile - 1) / a.sys_tile));
    hipLaunchKernelGGL((k_dirac<Si, So, G, C, R>), grid, dim3(kThreads), 0, st, a);
    return hipGetLastError();
}

}  // namespace

// Supported combinations (spinor in, spinor out, links, clover, compute):
//   all FP64; all FP32; FP16/BF16 spinors and links with FP32 clover and
//   compute; FP32/FP16/BF16 input with FP64 output, links, clover and compute
//   (the FP64 operator applied to a low-precision preconditioned vector);
//   FP16/BF16 input with FP32 output, links, clover and compute.
hipError_t launch_dirac(const DiracArgs& a, Prec in_p, Prec out_p, Prec link_p, Prec clover_p, Prec compute,
                        hipStream_t st) {
    if (compute == P_F32) {  // 4^4 tiles: the tiled kernel of tm_sap.hip
        const hipError_t e = launch_dirac_44(a, in_p, out_p, link_p, clover_p, st);
        if (e != hipErrorNotSupported) return e;
    }
#define TM_CASE(PI, PO, PL, PC, PR, TI, TO, TL, TC, TR)                                      \
    if (in_p == PI && out_p == PO && link_p == PL && clover_p == PC && compute == PR) \
        return run<TI, TO, TL, TC, TR>(a, st);
    TM_CASE(P_F32, P_F32, P_F32, P_F32, P_F32, float, float, float, float, float)
    TM_CASE(P_F16, P_F16, P_F16, P_F32, P_F32, f16, f16, f16, float, float)
    TM_CASE(P_BF16, P_BF16, P_BF16, P_F32, P_F32, bf16, bf16, bf16, float, float)
    TM_CASE(P_F16, P_F32, P_F32, P_F32, P_F32, f16, float, float, float, float)
    TM_CASE(P_BF16, P_F32, P_F32, P_F32, P_F32, bf16, float, float, float, float)
#undef TM_CASE
    if (out_p == P_F64 && link_p == P_F64 && clover_p == P_F64 && compute == P_F64) {
        const int* lb = a.g.lb;
        const bool is44 = lb[0] == 4 && lb[1] == 4 && lb[2] == 4 && lb[3] == 4;
        const unsigned nwg = (unsigned)((a.g.V + kThreads - 1) / kThreads), rounds = (nwg + kCUs - 1) / kCUs;
        // Other tiles (their links stay in memory): one lane per site reads a site's clover once for all systems,
        // but holds one workgroup per compute unit, so its time goes in rounds of 256 of them.  It is taken where
        // these are at least 3/4 full, from 640 workgroups on or with six or more systems.  One lane against two,
        // 2 / 6 / 12 systems: 16^4 (256 workgroups) 37 / 83 / 162 us against 34 / 92 / 191, 18^3x14 (319) 54 / 135 / 275
        // against 40 / 107 / 230, 18^4 (411) 59 / 153 / 309 against 53 / 156 / 330, 20x22^2x20 (757) 105 / 295 / 573
        // against 117 / 350 / 672, 30^4 474 / 1167 / 2306 against 532 / 1480 / 2816.
        // One system gains nothing from the shared clover and takes it from 896 workgroups on with rounds 7/8 full: 20x22x24x26
        // (1073) 106 us against 103, 22^4 (916) 87 against 92, 30^4 314 against 320, 34^4 502 against 526.
        const unsigned slots = kCUs * rounds;
        const bool one_lane = is44            ? a.nsys > 1 && a.g.V * a.nsys > kSplitSites
                              : a.nsys == 1 ? nwg >= 896 && 8 * nwg >= 7 * slots
                                            : nwg >= kCUs && 4 * nwg >= 3 * slots && (nwg >= 640 || a.nsys >= 6);
        if (in_p == P_F64 && one_lane) {
            DiracArgs t = a;
            t.sys_tile = pick_sys_tile(nwg, a.nsys, kCUs, 0.4, true);
            const dim3 grid(nwg, (unsigned)((a.nsys + t.sys_tile - 1) / t.sys_tile));
            if (is44)
                hipLaunchKernelGGL(k_dirac_lk<true>, grid, dim3(kThreads), 0, st, t);
            else
                hipLaunchKernelGGL(k_dirac_lk<false>, grid, dim3(kThreads), 0, st, t);
            return hipGetLastError();
        }
        if (in_p == P_F64) return run_pair<FieldOf<double>, double>(a, st);
        if (in_p == P_F32) return run_pair<FieldOf<float>, double>(a, st);
        if (in_p == P_F16) return run_pair<FieldOf<f16>, double>(a, st);
        if (in_p == P_BF16) return run_pair<FieldOf<bf16>, double>(a, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_dirac_canonical(const DiracArgs& a, hipStream_t st) { return run_pair<Canonical, double>(a, st); }

}  // namespace tmsap
