// Spin algebra with two lanes per site.
//
// Lane c (0 or 1) of a site's pair (adjacent lanes of a wavefront) owns
// chirality c of every site vector: spins (0, 1) for c = 0, spins (2, 3) for
// c = 1, six complex numbers.  The clover term and the site inverses are block
// diagonal in chirality, so each lane applies its own 6x6 block.  A hop works
// on a half spinor of two colour vectors h_0, h_1 (tm_device.h); lane c forms
// h_c from spin c of the neighbour and the lower spin that gamma_mu pairs with
// it, multiplies it by the link, and keeps three colour accumulators: `up`
// (spin c), `same` (lower spin 2 + c, directions t and z) and `cross` (lower
// spin 3 - c, directions x and y).  One exchange between the two lanes after
// the last hop turns these back into the chirality-owned form.
//
// Per lane this halves the registers of one site per lane, which is what the
// FP64 and the even-odd Schwarz kernels are short of.
#pragma once

#include "tm_device.h"
#include "tm_reduce.h"

namespace tmsap {

// value of the other lane of the pair (DPP quad_perm [1,0,3,2])
__device__ inline float pair_swap(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xb1, 0xf, 0xf, true));
}
__device__ inline double pair_swap(double v) {
    const long long b = __builtin_bit_cast(long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0xb1, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0xb1, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (long long)(((unsigned long long)hi << 32) | lo));
}
template <class R> __device__ inline cplx<R> pair_swap(cplx<R> v) { return cmk(pair_swap(v.re), pair_swap(v.im)); }
template <class R> __device__ inline cplx<R> pick(bool a, cplx<R> x, cplx<R> y) {
    return cmk(a ? x.re : y.re, a ? x.im : y.im);
}

// A colour vector, and a chirality-owned site vector (two spins).
template <class R> struct Col {
    cplx<R> v[3];
};
template <class R> struct Chir {
    cplx<R> v[6];
};

// An index the compiler cannot see through: what is read or computed from it stays where it is
// written, instead of being hoisted out of the system and MR loops (the link reads above all, which
// do not change there) and spilled.
__device__ inline int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Keeps a formed vector formed: without it the compiler moves the arithmetic down to the vector's use
// and holds everything it is formed from until then.
template <class R> __device__ inline void pin(Col<R>& v) {
#pragma unroll
    for (int k = 0; k < 3; ++k) asm volatile("" : "+v"(v.v[k].re), "+v"(v.v[k].im));
}

// Before a store: at this register pressure ROCm 7.2's compiler has put a store's address into registers
// that still held part of its data (x read as 16-byte pieces, updated, and stored as those pieces).
template <class R> __device__ inline void pin(Chir<R>& v) {
#pragma unroll
    for (int k = 0; k < 6; ++k) asm volatile("" : "+v"(v.v[k].re), "+v"(v.v[k].im));
}

// Directions whose partner of spin c is 3 - c (else 2 + c).
__host__ __device__ constexpr bool pair_cross(int mu) { return mu == 1 || mu == 2; }

// h_c = p -+ (B_mu lower)_c for p = spin c and q = its partner; s = 2 c - 1.
// DIR +1: forward hop (1 - gamma_mu), -1: backward (1 + gamma_mu).
template <int MU, int DIR, class R>
__device__ inline void pair_project(const Col<R>& p, const Col<R>& q, R s, Col<R>& h) {
    const R f = DIR > 0 ? (R)1 : (R)-1, fs = DIR > 0 ? -s : s;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const cplx<R> a = p.v[k], b = q.v[k];
        if constexpr (MU == 0) h.v[k] = cmk(a.re + f * b.re, a.im + f * b.im);
        if constexpr (MU == 1) h.v[k] = cmk(a.re - f * b.im, a.im + f * b.re);
        if constexpr (MU == 2) h.v[k] = cmk(a.re + fs * b.re, a.im + fs * b.im);
        if constexpr (MU == 3) h.v[k] = cmk(a.re - fs * b.im, a.im + fs * b.re);
    }
}

template <class R> struct PairAcc {
    Col<R> up, same, cross;
};

template <class R> __device__ inline void pin(PairAcc<R>& a) {
    pin(a.up);
    pin(a.same);
    pin(a.cross);
}

template <class R> __device__ inline void pair_zero(PairAcc<R>& a) {
#pragma unroll
    for (int k = 0; k < 3; ++k) a.up.v[k] = a.same.v[k] = a.cross.v[k] = cmk<R>(0, 0);
}

// Adds the finished product g_c of one hop: spin c takes g, its partner the
// lift -+ (B_mu^+ g).
template <int MU, int DIR, class R>
__device__ inline void pair_accumulate(const Col<R>& g, R s, PairAcc<R>& a) {
    const R f = DIR > 0 ? (R)1 : (R)-1, fs = DIR > 0 ? s : -s;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const cplx<R> t = g.v[k];
        a.up.v[k] = a.up.v[k] + t;
        if constexpr (MU == 0) a.same.v[k] = cmk(a.same.v[k].re + f * t.re, a.same.v[k].im + f * t.im);
        if constexpr (MU == 1) a.cross.v[k] = cmk(a.cross.v[k].re + f * t.im, a.cross.v[k].im - f * t.re);
        if constexpr (MU == 2) a.cross.v[k] = cmk(a.cross.v[k].re - fs * t.re, a.cross.v[k].im - fs * t.im);
        if constexpr (MU == 3) a.same.v[k] = cmk(a.same.v[k].re - fs * t.im, a.same.v[k].im + fs * t.re);
    }
}

// The hop sum in chirality-owned form: lane 0 gets spins 0 and 1, lane 1 spins 2 and 3.
template <class R> __device__ inline void pair_finish(const PairAcc<R>& a, bool lower, Chir<R>& out) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const cplx<R> r1 = pair_swap(pick(lower, a.up.v[k], a.same.v[k]));  // lane 0: spin 1, lane 1: spin 2's half
        const cplx<R> r2 = pair_swap(a.cross.v[k]);
        out.v[k] = pick(lower, r1 + a.cross.v[k], a.up.v[k]);
        out.v[3 + k] = pick(lower, r2 + a.same.v[k], r1);
    }
}

// Spin c and its partner of direction MU from the chirality-owned vectors of the pair.
template <int MU, class R>
__device__ inline void pair_spins(const Chir<R>& v, bool lower, Col<R>& p, Col<R>& q) {
    constexpr bool cross = pair_cross(MU);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const cplx<R> first = v.v[k], second = v.v[3 + k];
        // lane 0 gives spin 1; lane 1 gives lane 0's partner: spin 2, or 3 across
        const cplx<R> got = pair_swap(cross ? second : pick(lower, first, second));
        p.v[k] = pick(lower, got, first);
        q.v[k] = pick(lower, cross ? first : second, got);
    }
}

// Complex products in FP64 as fused multiply-adds written out: where a product could be fused with either of two
// sums the compiler chooses by what surrounds it, and two kernels would round one system's result differently.
// The choices here are its own for each expression by itself: of those tried nearest to the same operator by
// torch (2.08e-16 on 16^4; with the other product of each pair fused 2.09, third rows as one chain of four 2.10).
__device__ inline double fuse(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ inline cplx<double> mul_fixed(cplx<double> a, cplx<double> b) {  // a b
    return cmk(fuse(a.re, b.re, -(a.im * b.im)), fuse(a.im, b.re, a.re * b.im));
}
__device__ inline cplx<double> dag_fixed(cplx<double> a, cplx<double> b) {  // conj(a) b
    return cmk(fuse(a.re, b.re, a.im * b.im), fuse(a.re, b.im, -(a.im * b.re)));
}
__device__ inline cplx<double> mad_fixed(cplx<double> a, cplx<double> b, cplx<double> c) {  // a b + c
    return cmk(fuse(-a.im, b.im, fuse(a.re, b.re, c.re)), fuse(a.im, b.re, fuse(a.re, b.im, c.im)));
}
__device__ inline cplx<double> dagmad_fixed(cplx<double> a, cplx<double> b, cplx<double> c) {  // conj(a) b + c
    return cmk(fuse(a.im, b.im, fuse(a.re, b.re, c.re)), fuse(-a.im, b.re, fuse(a.re, b.im, c.im)));
}
__device__ inline cplx<double> cross_fixed(cplx<double> a, cplx<double> b, cplx<double> c, cplx<double> d) {
    return conj(mul_fixed(a, b) - mul_fixed(c, d));  // conj(a b - c d)
}

// g = U h and g = U^+ h for one colour vector; U from its first two rows u (row-major).
template <class R> __device__ inline void pair_mul(const cplx<R> u[6], const Col<R>& h, Col<R>& g) {
    const cplx<R> a = conj(u[1] * u[5] - u[2] * u[4]), b = conj(u[2] * u[3] - u[0] * u[5]),
                  c = conj(u[0] * u[4] - u[1] * u[3]);
    g.v[0] = cmad(u[2], h.v[2], cmad(u[1], h.v[1], u[0] * h.v[0]));
    g.v[1] = cmad(u[5], h.v[2], cmad(u[4], h.v[1], u[3] * h.v[0]));
    g.v[2] = cmad(c, h.v[2], cmad(b, h.v[1], a * h.v[0]));
}
template <class R> __device__ inline void pair_dag_mul(const cplx<R> u[6], const Col<R>& h, Col<R>& g) {
    const cplx<R> r[3] = {conj(u[1] * u[5] - u[2] * u[4]), conj(u[2] * u[3] - u[0] * u[5]),
                          conj(u[0] * u[4] - u[1] * u[3])};
#pragma unroll
    for (int i = 0; i < 3; ++i)
        g.v[i] = cjmad(r[i], h.v[2], cjmad(u[3 + i], h.v[1], conj(u[i]) * h.v[0]));
}
// The same in FP64 with a fixed rounding.
__device__ inline void pair_mul_fixed(const cplx<double> u[6], const Col<double>& h, Col<double>& g) {
    const cplx<double> r[9] = {u[0], u[1], u[2], u[3], u[4], u[5], cross_fixed(u[1], u[5], u[2], u[4]),
                               cross_fixed(u[2], u[3], u[0], u[5]), cross_fixed(u[0], u[4], u[1], u[3])};
#pragma unroll
    for (int i = 0; i < 3; ++i)
        g.v[i] = mad_fixed(r[3 * i + 2], h.v[2], mad_fixed(r[3 * i + 1], h.v[1], mul_fixed(r[3 * i], h.v[0])));
}
__device__ inline void pair_dag_mul_fixed(const cplx<double> u[6], const Col<double>& h, Col<double>& g) {
    const cplx<double> r[3] = {cross_fixed(u[1], u[5], u[2], u[4]), cross_fixed(u[2], u[3], u[0], u[5]),
                               cross_fixed(u[0], u[4], u[1], u[3])};
#pragma unroll
    for (int i = 0; i < 3; ++i)
        g.v[i] = dagmad_fixed(r[i], h.v[2], dagmad_fixed(u[3 + i], h.v[1], dag_fixed(u[i], h.v[0])));
}

// Plane k of a field of V units per plane: the same address for every lane, so that the planes of one
// site share one per-lane index.
template <class S> __device__ inline const void* plane(const void* base, int k, long long V) {
    return static_cast<const char*>(base) + (size_t)k * V * Unit<S>::bytes;
}
template <class S> __device__ inline void* plane(void* base, int k, long long V) {
    return static_cast<char*>(base) + (size_t)k * V * Unit<S>::bytes;
}

// Chirality c of a site: units 3c .. 3c + 2 of the spinor layout.
template <class R, class S>
__device__ inline void load_chir(const void* base, const float* scale, long long V, long long s, int c, Chir<R>& p) {
    R u[4];
    const size_t at = (size_t)(3 * c) * V + s;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        Unit<S>::load(plane<S>(base, k, V), at, u);
        p.v[2 * k] = cmk(u[0], u[1]);
        p.v[2 * k + 1] = cmk(u[2], u[3]);
    }
    if constexpr (HasScale<S>::value) {
        const R sc = (R)scale[s];
#pragma unroll
        for (int i = 0; i < 6; ++i) p.v[i] = sc * p.v[i];
    }
}

// Both lanes of the pair must be active (the FP16 scale spans the site).
template <class R, class S>
__device__ inline void store_chir(void* base, float* scale, long long V, long long s, int c, const Chir<R>& p) {
    const size_t at = (size_t)(3 * c) * V + s;
    if constexpr (HasScale<S>::value) {
        float m = 0.f;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            m = fmaxf(m, fabsf((float)p.v[i].re));
            m = fmaxf(m, fabsf((float)p.v[i].im));
        }
        m = fmaxf(m, pair_swap(m));
        float sc;
        const int e = fp16_site_exponent(m, &sc);
        if (c == 0) scale[s] = sc;
        const bool zero = sc == 0.f;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            float u[4] = {(float)p.v[2 * k].re, (float)p.v[2 * k].im, (float)p.v[2 * k + 1].re,
                          (float)p.v[2 * k + 1].im};
#pragma unroll
            for (int q = 0; q < 4; ++q) u[q] = zero ? u[q] * 0.f : ldexpf(u[q], -e);  // NaN stays NaN
            Unit<S>::store(plane<S>(base, k, V), at, u);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const R u[4] = {p.v[2 * k].re, p.v[2 * k].im, p.v[2 * k + 1].re, p.v[2 * k + 1].im};
            Unit<S>::store(plane<S>(base, k, V), at, u);
        }
    }
}

// A field of spinors: a site's chirality c, and the two spins that lane c needs of a neighbour.
template <class S> struct FieldOf {  // internal layout, units of four reals
    const void* base;
    const float* scale;
    long long V;
    __device__ inline FieldOf(const void* p, const float* sc, int sys, const Geo& g) : FieldOf(p, sc, sys, g.V) {}
    __device__ inline FieldOf(const void* p, const float* sc, int sys, long long sites)
        : base(static_cast<const char*>(p) + (size_t)sys * 6 * sites * Unit<S>::bytes),
          scale(sc ? sc + (size_t)sys * sites : nullptr), V(sites) {}
    __device__ inline void chirality(long long s, int c, Chir<double>& v) const {
        load_chir<double, S>(base, scale, V, s, c, v);
    }
    struct Raw {
        Chir<double> v;
    };
    template <int MU> __device__ inline void read(long long s, int c, Raw& r) const { chirality(s, c, r.v); }
    template <int MU> static __device__ inline void spins(const Raw& r, int c, Col<double>& p, Col<double>& q) {
        pair_spins<MU>(r.v, c != 0, p, q);
    }
    static constexpr bool kCanonical = false;
};

// The two rows of the FP64 link MU of a site, which both lanes of the pair need: each loads one complex number
// of every unit, 1 KiB in a row per wavefront, and takes the other from its partner.  All lanes active.
template <int MU>
__device__ inline void link_read(const void* links, long long V, long long site, int c, cplx<double> u[6]) {
    double2 w[3];
#pragma unroll
    for (int q = 0; q < 3; ++q)
        w[q] = static_cast<const double2*>(plane<double>(links, 3 * MU + q, V))[2 * (size_t)site + c];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        u[2 * q] = cmk(dpp_v<0xa0, 0xf>(w[q].x), dpp_v<0xa0, 0xf>(w[q].y));      // the even lane's
        u[2 * q + 1] = cmk(dpp_v<0xf5, 0xf>(w[q].x), dpp_v<0xf5, 0xf>(w[q].y));  // the odd lane's
    }
}

}  // namespace tmsap
