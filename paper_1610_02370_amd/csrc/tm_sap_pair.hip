// Half-sweeps of the Schwarz smoother (section 2.4) on 4^4 blocks with two
// lanes per site (tm_pair.h): the FP64 smoother, and the smoother with
// even-odd preconditioned block solves (section 2.5) at every precision.
//
// With one lane per site both run out of registers (the FP64 clover alone
// takes 144; the even-odd solve adds the site inverses to the clover), and the
// even-odd solve leaves half of the lanes idle in every step.  Two lanes per
// site each hold one chirality's 6x6 blocks and vectors.  A block's links sit
// in LDS (two rows, third rebuilt on use), read by both lanes of a pair as one
// broadcast; the vector being multiplied is exchanged through LDS.
//
// LDS rows are padded so that the two lanes of a pair, which read rows three
// apart, fall on different banks: a row stride of 8 mod 16 entries in FP64 and
// 16 mod 32 in FP32 puts them 128 bytes apart.
#include <type_traits>

#include "tm_internal.h"
#include "tm_pair.h"
#include "tm_reduce.h"
#include "tm_sap_index.h"

namespace tmsap {

namespace {

constexpr int kSites = 256;  // of a block

// Row strides for vectors over a block's sites and over one parity's.
template <class R> struct Pad {
    static constexpr int full = sizeof(R) == 8 ? 264 : 272, half = sizeof(R) == 8 ? 136 : 144;
};

// log2 of the local-index stride of direction mu (t, x, y, z) and its axis.
__host__ __device__ constexpr int dir_shift(int mu) { return mu == 0 ? 6 : 2 * (mu - 1); }
__host__ __device__ constexpr int dir_axis(int mu) { return mu == 0 ? 0 : 4 - mu; }

// Local coordinate of site l along mu, and the halo column of a face site: axis * 64 + its position,
// lexicographic over the other three axes (as S44Site's fsrc / bsrc).
template <int MU> __device__ inline int loc(int l) { return (l >> dir_shift(MU)) & 3; }
template <int MU> __device__ inline int face_col(int l) {
    constexpr int sh = dir_shift(MU);
    return dir_axis(MU) * 64 + (((l >> (sh + 2)) << sh) | (l & ((1 << sh) - 1)));
}

__device__ inline cplx<double> lds_get(const cplx<double>* p) {
    const double2 t = *reinterpret_cast<const double2*>(p);
    return cmk(t.x, t.y);
}
__device__ inline cplx<float> lds_get(const cplx<float>* p) {
    const float2 t = *reinterpret_cast<const float2*>(p);
    return cmk(t.x, t.y);
}
__device__ inline void lds_set(cplx<double>* p, cplx<double> v) { *reinterpret_cast<double2*>(p) = make_double2(v.re, v.im); }
__device__ inline void lds_set(cplx<float>* p, cplx<float> v) { *reinterpret_cast<float2*>(p) = make_float2(v.re, v.im); }

// Rows 6c .. 6c + 5 of a vector [12][stride]: chirality c of column n.
template <int ST, class R> __device__ inline void vec_put(cplx<R>* xs, int n, int c, const Chir<R>& v) {
#pragma unroll
    for (int i = 0; i < 6; ++i) lds_set(xs + (6 * c + i) * ST + n, v.v[i]);
}

// Links in LDS in 16-byte units: FP64 one complex each, [4 mu][6][256]; FP32 two, [4 mu][3][256].
template <class R> struct LinkLds;
template <> struct LinkLds<double> {
    double2 u[24][kSites];
    __device__ inline void put(int mu, int q, int n, const double v[4]) {
        u[6 * mu + 2 * q][n] = make_double2(v[0], v[1]);
        u[6 * mu + 2 * q + 1][n] = make_double2(v[2], v[3]);
    }
    __device__ inline void get(int mu, int n, cplx<double> o[6]) const {
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const double2 t = u[6 * mu + k][n];
            o[k] = cmk(t.x, t.y);
        }
    }
};
template <> struct LinkLds<float> {
    float4 u[12][kSites];
    __device__ inline void put(int mu, int q, int n, const float v[4]) {
        u[3 * mu + q][n] = make_float4(v[0], v[1], v[2], v[3]);
    }
    __device__ inline void get(int mu, int n, cplx<float> o[6]) const {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float4 t = u[3 * mu + k][n];
            o[2 * k] = cmk(t.x, t.y);
            o[2 * k + 1] = cmk(t.z, t.w);
        }
    }
};

// Column of site l's links.  CS 1 (lanes on the sites of one parity): the even sites' links first, then
// the odd sites', so that a wavefront reads consecutive columns.
__device__ inline int parity_of(int l) { return (l ^ (l >> 2) ^ (l >> 4) ^ (l >> 6)) & 1; }
template <int CS> __device__ inline int link_col(int l) { return CS ? (l >> 1) | (parity_of(l) << 7) : l; }

// The block's links: unit u = 3 mu + q of every site, NT threads; read into registers, then put in LDS.
template <class R, int NT> struct LinkRegs {
    R v[12 * kSites / NT][4];
};
template <class R, class G, int NT>
__device__ inline void read_links(const void* links, long long V, long long s0, int tid, LinkRegs<R, NT>& r) {
#pragma unroll
    for (int i = 0; i < 12 * kSites / NT; ++i) {
        const int e = i * NT + tid;
        Unit<G>::load(links, (size_t)(e >> 8) * V + s0 + (e & 255), r.v[i]);
    }
}
template <int CS, class R, int NT>
__device__ inline void put_links(const LinkRegs<R, NT>& r, int tid, LinkLds<R>& lk) {
#pragma unroll
    for (int i = 0; i < 12 * kSites / NT; ++i) {
        const int e = i * NT + tid, u = e >> 8;
        lk.put(u / 3, u % 3, link_col<CS>(e & 255), r.v[i]);
    }
}

// The two hops along MU of site l inside the block, its neighbours in columns n >> CS of xs.  A
// neighbour outside the block is column kSites >> CS, which holds zeros (and any link): without
// branches the compiler can have the next hop's LDS reads in flight while it works on this one.
template <int MU, int ST, int CS, class R>
__device__ inline void hops_mu(const cplx<R>* xs, const LinkLds<R>& lk, int l, int par, int c, R s,
                               PairAcc<R>& acc) {
    constexpr int str = 1 << dir_shift(MU);
    const int rq = pair_cross(MU) ? 9 - 3 * c : 6 + 3 * c;
    const int L = loc<MU>(l);
    {
        const int n = (L < 3 ? l + str : kSites) >> CS;
        Col<R> p, q, h, g;
        cplx<R> u[6];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            p.v[k] = lds_get(xs + (3 * c + k) * ST + n);
            q.v[k] = lds_get(xs + (rq + k) * ST + n);
        }
        lk.get(MU, CS ? (l >> 1) | (par << 7) : l, u);
        pair_project<MU, +1>(p, q, s, h);
        pair_mul(u, h, g);
        pair_accumulate<MU, +1>(g, s, acc);
    }
    {
        const int n = (L > 0 ? l - str : kSites) >> CS;
        Col<R> p, q, h, g;
        cplx<R> u[6];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            p.v[k] = lds_get(xs + (3 * c + k) * ST + n);
            q.v[k] = lds_get(xs + (rq + k) * ST + n);
        }
        const int m = L > 0 ? l - str : l;
        lk.get(MU, CS ? (m >> 1) | ((par ^ 1) << 7) : m, u);
        pair_project<MU, -1>(p, q, s, h);
        pair_dag_mul(u, h, g);
        pair_accumulate<MU, -1>(g, s, acc);
    }
}

// acc += the in-block hops of site l (of parity `par`, which only CS 1 uses).
template <int ST, int CS, class R>
__device__ inline void hops(const cplx<R>* xs, const LinkLds<R>& lk, int l, int par, int c, R s, PairAcc<R>& acc) {
    l = opaque(l);
    hops_mu<0, ST, CS>(xs, lk, l, par, c, s, acc);
    hops_mu<1, ST, CS>(xs, lk, l, par, c, s, acc);
    hops_mu<2, ST, CS>(xs, lk, l, par, c, s, acc);
    hops_mu<3, ST, CS>(xs, lk, l, par, c, s, acc);
    pin(acc);
}

// One halo duty (entry e = axis * 64 + position, axis the same for the wavefront).  The reads are
// issued together with the block's other reads, so that a block pays one memory latency; what they
// become is formed later: of the site above the upper face the projected colour vector h_c, of the
// site below the lower face the product U^+ h_c, boundary phases applied.
template <class R> struct Halo {
    Chir<R> up, dn;
    cplx<R> u[6];
    bool up_wrap, dn_wrap;
};
template <class S, class G, class R>
__device__ inline void halo_read(const Geo& g, const void* links, const void* xx, const float* xsc, const int B[4],
                                 long long blk, int e, int c, Halo<R>& t) {
    S44Site ix;
    s44_lane(g, B, blk, opaque(e), ix);
    const int axis = __builtin_amdgcn_readfirstlane(e >> 6), mu = axis == 0 ? 0 : 4 - axis;
    t.up_wrap = ix.up_wrap;
    t.dn_wrap = ix.dn_wrap;
    load_chir<R, S>(xx, xsc, g.V, ix.dn_site, c, t.dn);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        R w[4];
        Unit<G>::load(plane<G>(links, 3 * mu + q, g.V), (size_t)ix.dn_site, w);
        t.u[2 * q] = cmk(w[0], w[1]);
        t.u[2 * q + 1] = cmk(w[2], w[3]);
    }
    load_chir<R, S>(xx, xsc, g.V, ix.up_site, c, t.up);
}

template <int MU, class R>
__device__ inline void halo_mu(const Geo& g, const Halo<R>& t, int c, R s, Col<R>& up, Col<R>& dn) {
    const R pr = sizeof(R) == 4 ? (R)g.bcrf[MU] : (R)g.bcr[MU], pi = sizeof(R) == 4 ? (R)g.bcif[MU] : (R)g.bci[MU];
    Col<R> p, q, h;
    pair_spins<MU>(t.dn, c != 0, p, q);
    pair_project<MU, -1>(p, q, s, h);
    if (t.dn_wrap) {
#pragma unroll
        for (int k = 0; k < 3; ++k) h.v[k] = cmk(pr, -pi) * h.v[k];
    }
    pair_dag_mul(t.u, h, dn);
    pair_spins<MU>(t.up, c != 0, p, q);
    pair_project<MU, +1>(p, q, s, up);
    if (t.up_wrap) {
#pragma unroll
        for (int k = 0; k < 3; ++k) up.v[k] = cmk(pr, pi) * up.v[k];
    }
}

template <class R>
__device__ inline void halo_form(const Geo& g, const Halo<R>& t, int e, int c, R s, Col<R>& up, Col<R>& dn) {
    switch (__builtin_amdgcn_readfirstlane(e >> 6)) {
        case 0: halo_mu<0>(g, t, c, s, up, dn); break;
        case 1: halo_mu<3>(g, t, c, s, up, dn); break;
        case 2: halo_mu<2>(g, t, c, s, up, dn); break;
        default: halo_mu<1>(g, t, c, s, up, dn); break;
    }
    pin(up);
    pin(dn);
}

// Halo entries in the columns of vectors (CS 1: of the odd sites' vector, then the even sites'):
// rows 3c + k the products from below, 6 + 3c + k the vectors from above.
template <int ST, int CS> __device__ inline int halo_col(int e) { return CS ? (e & 1) * 12 * ST + (e >> 1) : e; }
template <int ST, int CS, class R>
__device__ inline void halo_put(cplx<R>* xs, int e, int c, const Col<R>& up, const Col<R>& dn) {
    xs += halo_col<ST, CS>(e);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        lds_set(xs + (3 * c + k) * ST, dn.v[k]);
        lds_set(xs + (6 + 3 * c + k) * ST, up.v[k]);
    }
}

template <int MU, int ST, int CS, class R>
__device__ inline void halo_hops_mu(const cplx<R>* xs, const LinkLds<R>& lk, int l, int c, R s, PairAcc<R>& acc) {
    const int L = loc<MU>(l), col = halo_col<ST, CS>(face_col<MU>(l));
    __builtin_amdgcn_sched_barrier(0);
    if (L == 3) {
        Col<R> h, g;
        cplx<R> u[6];
        lk.get(MU, link_col<CS>(l), u);
#pragma unroll
        for (int k = 0; k < 3; ++k) h.v[k] = lds_get(xs + (6 + 3 * c + k) * ST + col);
        pair_mul(u, h, g);
        pair_accumulate<MU, +1>(g, s, acc);
    }
    if (L == 0) {
        Col<R> g;
#pragma unroll
        for (int k = 0; k < 3; ++k) g.v[k] = lds_get(xs + (3 * c + k) * ST + col);
        pair_accumulate<MU, -1>(g, s, acc);
    }
}

template <int ST, int CS, class R>
__device__ inline void halo_hops(const cplx<R>* xs, const LinkLds<R>& lk, int l, int c, R s, PairAcc<R>& acc) {
    l = opaque(l);
    halo_hops_mu<0, ST, CS>(xs, lk, l, c, s, acc);
    halo_hops_mu<1, ST, CS>(xs, lk, l, c, s, acc);
    halo_hops_mu<2, ST, CS>(xs, lk, l, c, s, acc);
    halo_hops_mu<3, ST, CS>(xs, lk, l, c, s, acc);
}

// Lane c's chirality block of the packed clover.
template <class R, class C>
__device__ inline void load_clover_chir(const void* clover, long long V, long long s, int c, R A[36]) {
    const size_t at = (size_t)(9 * c) * V + s;
#pragma unroll
    for (int k = 0; k < 9; ++k) Unit<C>::load(plane<C>(clover, k, V), at, A + 4 * k);
}

// MR sums <q, rho>, <q, q> of the lane's chirality, one fused multiply-add per product.
template <class R>
__device__ inline void chir_dots(const Chir<R>& q, const Chir<R>& rho, R& qr_re, R& qr_im, R& qq) {
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        qr_re = qr_re + q.v[i].re * rho.v[i].re;
        qr_re = qr_re + q.v[i].im * rho.v[i].im;
        qr_im = qr_im + q.v[i].re * rho.v[i].im;
        qr_im = qr_im - q.v[i].im * rho.v[i].re;
        qq = qq + q.v[i].re * q.v[i].re;
        qq = qq + q.v[i].im * q.v[i].im;
    }
}

template <class R>
__device__ inline void chir_axpy(cplx<R> a, const Chir<R>& x, Chir<R>& y) {
#pragma unroll
    for (int i = 0; i < 6; ++i) y.v[i] = cmad(a, x.v[i], y.v[i]);
}

__device__ inline void block_coords(const Geo& g, int colour, int B[4]) {
    s44_block(g, colour, xcd_swizzle(blockIdx.x, gridDim.x), B);
#pragma unroll
    for (int q = 0; q < 4; ++q) B[q] = __builtin_amdgcn_readfirstlane(B[q]);
}

// What of x the half-sweep finds: nothing yet (r = b), nothing on its own colour (the halo hops alone),
// or all of it.  A template parameter: as run-time flags the compiler spilled what the branches leave
// unset.
enum { kFromZero = 0, kHaloOnly = 1, kFull = 2 };

// ---------------------------------------------------------------------------
// FP64 half-sweep: 512 threads per block, two wavefronts per SIMD, one
// workgroup per compute unit (146 KiB of LDS: links 96, exchange 50).
// 32^3x64, one system: 770 us per half-sweep (825 in bench.py's sweeps) against
// 1176 with one lane per site (376 bytes per lane of scratch, one wavefront per
// SIMD).  75 us of it per MR step (4.7 us per block, 2 wavefronts x 1084 vector
// instructions per SIMD); the other 470 us read 516 KB per block, which no second
// workgroup overlaps: 2.1 GB per half-sweep, 4.5 TB/s while it lasts.
constexpr int kPlain = 2 * kSites;

template <class S, class G, class C, class R, int MODE>
__global__ void __launch_bounds__(kPlain) __attribute__((amdgpu_waves_per_eu(2, 2))) k_sap_pair(SapArgs a) {
    constexpr int ST = Pad<R>::full;
    __shared__ __align__(16) cplx<R> xs[12 * ST];
    __shared__ __align__(16) LinkLds<R> lk;
    __shared__ R red[4 * kPlain / 64];
    const Geo& g = a.g;
    const int tid = threadIdx.x, l = tid >> 1, c = tid & 1;
    const bool lower = c != 0;
    const R s = lower ? (R)1 : (R)-1;
    int B[4];
    block_coords(g, a.colour, B);
    const long long blk = s44_block_index(g, B), s0 = blk * kSites;
    const int parity = parity_of(l);  // the block's own coordinates are even

    const size_t stride = (size_t)6 * g.V * Unit<S>::bytes;
    const int sys_begin = blockIdx.y * a.sys_tile;
    const int sys_end = min(a.nsys, sys_begin + a.sys_tile);
    Chir<R> x, rho;
    Halo<R> hl;
    auto read_system = [&](int sys) {
        const void* xx = reinterpret_cast<const char*>(a.x) + sys * stride;
        const float* xsc = a.x_scale ? a.x_scale + (size_t)sys * g.V : nullptr;
#pragma unroll
        for (int i = 0; i < 6; ++i) x.v[i] = cmk<R>(0, 0);
        if constexpr (MODE == kFull) load_chir<R, S>(xx, xsc, g.V, s0 + opaque(l), c, x);
        if constexpr (MODE != kFromZero) halo_read<S, G, R>(g, a.links, xx, xsc, B, blk, l, c, hl);
    };
    // b is read once the in-block hops are done: held through them it would spill
    auto read_b = [&](int sys) {
        load_chir<R, S>(reinterpret_cast<const char*>(a.b) + sys * stride,
                        a.b_scale ? a.b_scale + (size_t)sys * g.V : nullptr, g.V, s0 + opaque(l), c, rho);
    };

    // the block's reads issued together: one memory latency instead of one per kind (the clover, which
    // would not fit in registers beside them all, once the links are in LDS)
    LinkRegs<R, kPlain> lr;
    read_links<R, G>(a.links, g.V, s0, tid, lr);
    read_system(sys_begin);
    __builtin_amdgcn_sched_barrier(0);
    put_links<0>(lr, tid, lk);
    __builtin_amdgcn_sched_barrier(0);
    R A[36];
    load_clover_chir<R, C>(a.clover, g.V, s0 + l, c, A);
    if (tid < 12) lds_set(xs + tid * ST + kSites, cmk<R>(0, 0));
    __syncthreads();

    for (int sys = sys_begin;;) {
        const R mu = (R)(a.mu[sys] + g.mu_shift[parity]), tw = lower ? -mu : mu;
        if constexpr (MODE != kFromZero) {
            // r = b - D x: in-block hops, then the halo's colour vectors and the hops from them
            Col<R> up, dn;
            halo_form(g, hl, l, c, s, up, dn);
            PairAcc<R> acc;
            pair_zero(acc);
            if constexpr (MODE == kFull) {
                vec_put<ST>(xs, l, c, x);
                __syncthreads();
                hops<ST, 0>(xs, lk, l, 0, c, s, acc);
                __syncthreads();
            }
            read_b(sys);
            halo_put<ST, 0>(xs, l, c, up, dn);
            __syncthreads();
            halo_hops<ST, 0>(xs, lk, l, c, s, acc);
            Chir<R> t;
            pair_finish(acc, lower, t);
#pragma unroll
            for (int i = 0; i < 6; ++i)
                rho.v[i] = cmk(rho.v[i].re + (R)0.5 * t.v[i].re, rho.v[i].im + (R)0.5 * t.v[i].im);
            if constexpr (MODE == kFull) {
                clover_block_apply(A, tw, x.v, t.v);
#pragma unroll
                for (int i = 0; i < 6; ++i) rho.v[i] = rho.v[i] - t.v[i];
            }
            __syncthreads();
        } else {
            read_b(sys);
        }

        // minimal residual on D_BB from a zero correction, added to x as it goes
        for (int it = 0; it < a.mr_iters; ++it) {
            vec_put<ST>(xs, l, c, rho);
            __syncthreads();
            PairAcc<R> acc;
            pair_zero(acc);
            hops<ST, 0>(xs, lk, l, 0, c, s, acc);
            Chir<R> q;
            pair_finish(acc, lower, q);
#pragma unroll
            for (int i = 0; i < 6; ++i) q.v[i] = (R)-0.5 * q.v[i];
            clover_block_acc(A, tw, rho.v, q.v);
            R qr_re = 0, qr_im = 0, qq = 0;
            chir_dots(q, rho, qr_re, qr_im, qq);
            block_sum3(red, qr_re, qr_im, qq);
            if (qq >= min_normal<R>()) {
                const cplx<R> alpha = cmk(qr_re / qq, qr_im / qq);
                chir_axpy(alpha, rho, x);
                chir_axpy(-alpha, q, rho);
            }
        }
        pin(x);
        store_chir<R, S>(reinterpret_cast<char*>(a.x) + sys * stride,
                         a.x_scale ? a.x_scale + (size_t)sys * g.V : nullptr, g.V, s0 + opaque(l), c, x);
        if (++sys >= sys_end) break;
        read_system(sys);
    }
}

// ---------------------------------------------------------------------------
// Half-sweep with even-odd preconditioned block solves: 256 threads per block,
// two lanes per pair (2h, 2h+1) of an even and an odd site.  Every step of the
// reduced operator Dhat = D_oo - D_oe D_ee^-1 D_eo works on one parity, so a
// pair's lanes take its even site and its odd site in turn and none idles.
//   rhat_o = r_o - D_oe D_ee^-1 r_e,  MR on Dhat e_o = rhat_o from zero,
//   e_e = D_ee^-1 (r_e - D_eo e_o).
// The odd site's clover stays in registers, the even site's inverse through a
// system's MR steps.  75 KiB of LDS in FP32: two workgroups per compute unit.
// 32^3x64, +-mu in FP32: 890 us per half-sweep against 3690 with one lane per
// site; bound by vector issue (an MR step is 2100 instructions per wavefront, a
// fifth of them rebuilding third link rows).  Putting the links' reads, the
// first system's and the clover's in flight together, as the FP64 kernel does,
// spilled and cost 10 % here, where the other workgroup covers them.
constexpr int kEo = kSites;

// out = M v (adj: M^+ v) for a full 6x6 block.
template <class R>
__device__ inline void inverse_apply(const cplx<R> M[36], bool adj, const Chir<R>& v, Chir<R>& out) {
#pragma unroll
    for (int i = 0; i < 6; ++i) out.v[i] = cmk<R>(0, 0);
    if (adj) {
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int j = 0; j < 6; ++j) out.v[j] = cjmad(M[6 * i + j], v.v[i], out.v[j]);
    } else {
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int j = 0; j < 6; ++j) out.v[i] = cmad(M[6 * i + j], v.v[j], out.v[i]);
    }
}

template <class S, class G, class C, class R, int MODE>
__global__ void __launch_bounds__(kEo) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 8 ? 1 : 2)))
k_sap_pair_eo(SapArgs a) {
    constexpr int SH = Pad<R>::half;
    __shared__ __align__(16) cplx<R> xs[2 * 12 * SH];
    __shared__ __align__(16) LinkLds<R> lk;
    __shared__ R red[4 * kEo / 64];
    cplx<R>* const xo = xs;            // vectors on the odd sites, columns h
    cplx<R>* const xe = xs + 12 * SH;  // on the even sites
    const Geo& g = a.g;
    const int tid = threadIdx.x, h = tid >> 1, c = tid & 1;
    const bool lower = c != 0;
    const R s = lower ? (R)1 : (R)-1;
    int B[4];
    block_coords(g, a.colour, B);
    const long long blk = s44_block_index(g, B), s0 = blk * kSites;
    // parity of site 2h of the block (the block's own coordinates are even, and so is x there)
    const int odd0 = ((h >> 1) ^ (h >> 3) ^ (h >> 5)) & 1;
    const int le = 2 * h + odd0, lo = 2 * h + 1 - odd0;
    const long long half = g.V / 2, hh0 = s0 >> 1;


    const size_t stride = (size_t)6 * g.V * Unit<S>::bytes;
    const int sys_begin = blockIdx.y * a.sys_tile;
    const int sys_end = min(a.nsys, sys_begin + a.sys_tile);
    Chir<R> te, to, re, rho;
    Halo<R> hl[2];
    auto read_system = [&](int sys) {
        const void* xx = reinterpret_cast<const char*>(a.x) + sys * stride;
        const float* xsc = a.x_scale ? a.x_scale + (size_t)sys * g.V : nullptr;
        if constexpr (MODE == kFull) {
            load_chir<R, S>(xx, xsc, g.V, s0 + opaque(le), c, te);
            load_chir<R, S>(xx, xsc, g.V, s0 + opaque(lo), c, to);
        }
        if constexpr (MODE != kFromZero) {
#pragma unroll
            for (int k = 0; k < 2; ++k) halo_read<S, G, R>(g, a.links, xx, xsc, B, blk, 128 * k + h, c, hl[k]);
        }
    };
    auto read_b = [&](int sys) {  // after the in-block hops, as above
        const void* bb = reinterpret_cast<const char*>(a.b) + sys * stride;
        const float* bsc = a.b_scale ? a.b_scale + (size_t)sys * g.V : nullptr;
        load_chir<R, S>(bb, bsc, g.V, s0 + opaque(le), c, re);
        load_chir<R, S>(bb, bsc, g.V, s0 + opaque(lo), c, rho);
    };

    {
        LinkRegs<R, kEo> lr;
        read_links<R, G>(a.links, g.V, s0, tid, lr);
        put_links<1>(lr, tid, lk);
    }
    R A[36];
    load_clover_chir<R, C>(a.clover, g.V, s0 + lo, c, A);
    if (tid < 24) lds_set(xs + tid * SH + kSites / 2, cmk<R>(0, 0));
    __syncthreads();

    for (int sys = sys_begin;;) {
        const R me = (R)(a.mu[sys] + g.mu_shift[0]), mo = (R)(a.mu[sys] + g.mu_shift[1]);
        const R twe = lower ? -me : me, two = lower ? -mo : mo;
        const void* inv = a.eo_inv[a.eo_sel[sys]];
        const bool adj = (a.eo_adj >> sys) & 1ull;
        void* xx = reinterpret_cast<char*>(a.x) + sys * stride;
        float* xsc = a.x_scale ? a.x_scale + (size_t)sys * g.V : nullptr;
        read_system(sys);

        // ---- r = b - D x on both sites of the pair
        if constexpr (MODE != kFromZero) {
            Col<R> up[2], dn[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) halo_form(g, hl[k], 128 * k + h, c, s, up[k], dn[k]);
            PairAcc<R> ae, ao;
            pair_zero(ae);
            pair_zero(ao);
            if constexpr (MODE == kFull) {
                vec_put<SH>(xe, h, c, te);
                vec_put<SH>(xo, h, c, to);
                __syncthreads();
                hops<SH, 1>(xo, lk, le, 0, c, s, ae);
                hops<SH, 1>(xe, lk, lo, 1, c, s, ao);
                __syncthreads();
            }
            read_b(sys);
#pragma unroll
            for (int k = 0; k < 2; ++k) halo_put<SH, 1>(xs, 128 * k + h, c, up[k], dn[k]);
            __syncthreads();
            halo_hops<SH, 1>(xs, lk, le, c, s, ae);
            halo_hops<SH, 1>(xs, lk, lo, c, s, ao);
            Chir<R> t;
            pair_finish(ae, lower, t);
#pragma unroll
            for (int i = 0; i < 6; ++i) re.v[i] = cmk(re.v[i].re + (R)0.5 * t.v[i].re, re.v[i].im + (R)0.5 * t.v[i].im);
            pair_finish(ao, lower, t);
#pragma unroll
            for (int i = 0; i < 6; ++i)
                rho.v[i] = cmk(rho.v[i].re + (R)0.5 * t.v[i].re, rho.v[i].im + (R)0.5 * t.v[i].im);
            if constexpr (MODE == kFull) {
                clover_block_apply(A, two, to.v, t.v);
#pragma unroll
                for (int i = 0; i < 6; ++i) rho.v[i] = rho.v[i] - t.v[i];
                R Ae[36];
                load_clover_chir<R, C>(a.clover, g.V, s0 + le, opaque(c), Ae);
                clover_block_apply(Ae, twe, te.v, t.v);
#pragma unroll
                for (int i = 0; i < 6; ++i) re.v[i] = re.v[i] - t.v[i];
            }
            __syncthreads();
        } else {
            read_b(sys);
        }

        // the even site's inverse, read per system: held across the residual as well it would spill
        cplx<R> M[36];
        const size_t hm = (size_t)(18 * opaque(c)) * half + hh0 + h;
#pragma unroll
        for (int u = 0; u < 18; ++u) {
            R w[4];
            Unit<C>::load(plane<C>(inv, u, half), hm, w);
            M[2 * u] = cmk(w[0], w[1]);
            M[2 * u + 1] = cmk(w[2], w[3]);
        }

        // ---- rhat_o = r_o - D_oe (D_ee^-1 r_e)
        Chir<R> t, e;
        PairAcc<R> acc;
        inverse_apply(M, adj, re, t);
        vec_put<SH>(xe, h, c, t);
        __syncthreads();
        pair_zero(acc);
        hops<SH, 1>(xe, lk, lo, 1, c, s, acc);
        pair_finish(acc, lower, t);
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            rho.v[i] = cmk(rho.v[i].re + (R)0.5 * t.v[i].re, rho.v[i].im + (R)0.5 * t.v[i].im);
            e.v[i] = cmk<R>(0, 0);
        }

        // ---- MR on Dhat over the odd sites
        for (int it = 0; it < a.mr_iters; ++it) {
            vec_put<SH>(xo, h, c, rho);
            __syncthreads();
            // even: t_e = D_ee^-1 D_eo rho_o
            pair_zero(acc);
            hops<SH, 1>(xo, lk, le, 0, c, s, acc);
            Chir<R> u;
            pair_finish(acc, lower, u);
#pragma unroll
            for (int i = 0; i < 6; ++i) u.v[i] = (R)-0.5 * u.v[i];
            inverse_apply(M, adj, u, t);
            vec_put<SH>(xe, h, c, t);
            __syncthreads();
            // odd: q_o = D_oo rho_o - D_oe t_e
            pair_zero(acc);
            hops<SH, 1>(xe, lk, lo, 1, c, s, acc);
            Chir<R> q;
            pair_finish(acc, lower, q);
#pragma unroll
            for (int i = 0; i < 6; ++i) q.v[i] = (R)0.5 * q.v[i];
            clover_block_acc(A, two, rho.v, q.v);
            R qr_re = 0, qr_im = 0, qq = 0;
            chir_dots(q, rho, qr_re, qr_im, qq);
            block_sum3(red, qr_re, qr_im, qq);
            if (qq >= min_normal<R>()) {
                const cplx<R> alpha = cmk(qr_re / qq, qr_im / qq);
                chir_axpy(alpha, rho, e);
                chir_axpy(-alpha, q, rho);
            }
        }

        // ---- e_e = D_ee^-1 (r_e - D_eo e_o), x += e
        vec_put<SH>(xo, h, c, e);
        __syncthreads();
        pair_zero(acc);
        hops<SH, 1>(xo, lk, le, 0, c, s, acc);
        Chir<R> u;
        pair_finish(acc, lower, u);
#pragma unroll
        for (int i = 0; i < 6; ++i) u.v[i] = cmk(re.v[i].re + (R)0.5 * u.v[i].re, re.v[i].im + (R)0.5 * u.v[i].im);
        inverse_apply(M, adj, u, t);
        const long long he = s0 + opaque(le), ho = s0 + opaque(lo);
        if constexpr (MODE == kFull) {
            Chir<R> x;
            load_chir<R, S>(xx, xsc, g.V, he, c, x);
#pragma unroll
            for (int i = 0; i < 6; ++i) t.v[i] = t.v[i] + x.v[i];
            load_chir<R, S>(xx, xsc, g.V, ho, c, x);
#pragma unroll
            for (int i = 0; i < 6; ++i) e.v[i] = e.v[i] + x.v[i];
        }
        pin(t);
        pin(e);
        store_chir<R, S>(xx, xsc, g.V, he, c, t);
        store_chir<R, S>(xx, xsc, g.V, ho, c, e);
        if (++sys >= sys_end) break;
        __syncthreads();  // every read of xs done before the next system writes it
    }
}

template <class S, class G, class C, class R, int MODE>
void launch(const SapArgs& a, dim3 grid, hipStream_t st) {
    if (a.eo)
        hipLaunchKernelGGL((k_sap_pair_eo<S, G, C, R, MODE>), grid, dim3(kEo), 0, st, a);
    else if constexpr (sizeof(R) == 8)
        hipLaunchKernelGGL((k_sap_pair<S, G, C, R, MODE>), grid, dim3(kPlain), 0, st, a);
}

template <class S, class G, class C, class R>
hipError_t run(const SapArgs& args, hipStream_t st) {
    if (!args.eo && sizeof(R) == 4) return hipErrorNotSupported;  // FP32 arithmetic: k_sap_half_44
    SapArgs a = args;
    const long long n = (long long)a.g.nb[0] * a.g.nb[1] * a.g.nb[2] * a.g.nb[3] / 2;
    if (a.sys_tile <= 0) a.sys_tile = pick_sys_tile(n, a.nsys, (a.eo && sizeof(R) == 4 ? 2 : 1) * kCUs, 0.2, false);
    const dim3 grid((unsigned)n, (unsigned)((a.nsys + a.sys_tile - 1) / a.sys_tile));
    if (a.own_zero && a.halo_zero)
        launch<S, G, C, R, kFromZero>(a, grid, st);
    else if (a.own_zero)
        launch<S, G, C, R, kHaloOnly>(a, grid, st);
    else
        launch<S, G, C, R, kFull>(a, grid, st);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_sap_pair(const SapArgs& a, Prec sp, Prec lp, Prec cp, hipStream_t st) {
    const int* lb = a.g.lb;
    if (lb[0] != 4 || lb[1] != 4 || lb[2] != 4 || lb[3] != 4) return hipErrorNotSupported;
    if (sp == P_F64 && lp == P_F64 && cp == P_F64) return run<double, double, double, double>(a, st);
    if (sp == P_F32 && lp == P_F32 && cp == P_F32) return run<float, float, float, float>(a, st);
    if (sp == P_F16 && lp == P_F16 && cp == P_F32) return run<f16, f16, float, float>(a, st);
    if (sp == P_BF16 && lp == P_BF16 && cp == P_F32) return run<bf16, bf16, float, float>(a, st);
    return hipErrorNotSupported;
}

}  // namespace tmsap
