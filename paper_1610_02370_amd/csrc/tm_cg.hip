// Kernels of the even-odd reduced operator and of CG on its normal
// equations (the CG comparison of section 3, eq. (oereduced)).
//
// Vectors live on one parity: with the tile's x-extent even, the sites 2h and
// 2h+1 of the tiled layout are one even and one odd site, so a parity vector
// is a compact field [nsys][6 units][V/2] indexed by h = s / 2.  FP64 only:
// the CG is the plain FP64 baseline.
#include "tm_internal.h"
#include "tm_pair.h"
#include "tm_reduce.h"

namespace tmsap {

namespace {

constexpr int kThreads = 256;

__device__ inline int site_parity_tiled(const Geo& g, unsigned s) {
    const unsigned Vb = (unsigned)g.Vb;
    const unsigned blk = s / Vb;
    unsigned l = s - blk * Vb, tb = blk;
    int sum = 0;
#pragma unroll
    for (int a = 3; a >= 0; --a) {
        const unsigned lb = (unsigned)g.lb[a], nb = (unsigned)g.nb[a];
        const unsigned lq = l / lb, bq = tb / nb;
        sum += (int)(tb - bq * nb) * g.lb[a] + (int)(l - lq * lb);
        l = lq;
        tb = bq;
    }
    return sum & 1;
}

// A chunk's sum from its parts, pairwise.
template <int PARTS>
__device__ inline double sum_parts(const double* v) {
    return PARTS == 4 ? (v[0] + v[1]) + (v[2] + v[3]) : (PARTS == 2 ? v[0] + v[1] : v[0]);
}

// out_p = (D_pp^-1)? [ hop_sign * H in_hop + D_pp in_diag + add_sign * in_add ], H = -1/2 sum of hops
// between the parities, D_pp = (m+4) + clover + i mu Gamma5 on parity p; the Gamma5 flags multiply
// the hop input, the diagonal input and the output.  With `partials`, also ||out||^2 per workgroup and
// system.
//
// Two lanes per site (tm_pair.h), a run of 32 sites of one system per wavefront, the four wavefronts of a workgroup
// on `sys_tile` (1, 2 or 4) systems of the same sites.  Four runs make a chunk, whose sites stay together
// whatever the tile: a workgroup of tile 1 takes the four runs of chunks b, b + blocks, ..., one of tile 2 or 4 its
// part of them, two runs or one.  A system's sums therefore are the same bits in any number of systems: over a
// wavefront's runs first, then pairwise over the four wavefronts, in LDS or (sum_partials) from the parts.  Bound by the links and the site matrices: on 16^3x32,
// 126 MB (diagonal) to 150 MB (site inverse) per launch in 31-32 us, 4.0-4.8 TB/s, where a copy reaches 4.7;
// one lane per site kept that half lattice at one wavefront per SIMD and took 36 us.
template <int MU, bool G5HOP>
__device__ inline void parity_dir(const ParityArgs& a, const FieldOf<double>& in, unsigned s, const int nf[4],
                                  const int nbk[4], unsigned wrap, int c, double sg, PairAcc<double>& acc) {
    const Geo& g = a.g;
    __builtin_amdgcn_sched_barrier(0);  // one direction's operands live at a time
    cplx<double> uf[6], ub[6];
    FieldOf<double>::Raw pf, pb;
    in.read<MU>(nf[MU] >> 1, c, pf);
    link_read<MU>(a.links, g.V, s, c, uf);
    in.read<MU>(nbk[MU] >> 1, c, pb);
    link_read<MU>(a.links, g.V, nbk[MU], c, ub);
    Col<double> p, q, h, t;
    FieldOf<double>::spins<MU>(pf, c, p, q);
    if (G5HOP) {
#pragma unroll
        for (int k = 0; k < 3; ++k) q.v[k] = -q.v[k];
    }
    pair_project<MU, +1>(p, q, sg, h);
    if (wrap & (1u << MU)) {
#pragma unroll
        for (int k = 0; k < 3; ++k) h.v[k] = cmk(g.bcr[MU], g.bci[MU]) * h.v[k];
    }
    pair_mul(uf, h, t);
    pair_accumulate<MU, +1>(t, sg, acc);
    FieldOf<double>::spins<MU>(pb, c, p, q);
    if (G5HOP) {
#pragma unroll
        for (int k = 0; k < 3; ++k) q.v[k] = -q.v[k];
    }
    pair_project<MU, -1>(p, q, sg, h);
    if (wrap & (16u << MU)) {
#pragma unroll
        for (int k = 0; k < 3; ++k) h.v[k] = cmk(g.bcr[MU], -g.bci[MU]) * h.v[k];
    }
    pair_dag_mul(ub, h, t);
    pair_accumulate<MU, -1>(t, sg, acc);
    pin(acc);
    __builtin_amdgcn_sched_barrier(0);
}

template <bool HOP, bool DIAG, bool INV, bool G5HOP, int TILE>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) k_parity_op(ParityArgs a) {
    __shared__ double nrm[4];
    const Geo& g = a.g;
    const long long half = g.V / 2;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, c = lane & 1;
    const bool lower = c != 0;
    const double sg = lower ? 1.0 : -1.0;
    constexpr int runs = 4 / TILE;  // of a chunk, per system
    const int sys = blockIdx.y * TILE + w / runs;
    // block and part; a chunk's parts on one XCD (blocks is a multiple of 8)
    const int blocks = gridDim.x / TILE, row = blockIdx.x / 8u;
    const int part = row % TILE, first = blockIdx.x % 8u + 8 * (row / TILE);
    double n2 = 0;
    for (int vb = first; vb < a.chunks && sys < a.nsys; vb += blocks) {
        const long long at = (xcd_swizzle(vb, a.chunks) * 4 + part * runs + w % runs) * 32 + (lane >> 1);
        const bool on = at < half;
        const long long h = on ? at : 0;
        unsigned s = 2u * (unsigned)h;
        if (site_parity_tiled(g, s) != a.p) ++s;
        const double mu = a.mu_sign * (a.mu[sys] + g.mu_shift[a.p]);
        Chir<double> v;
#pragma unroll
        for (int i = 0; i < 6; ++i) v.v[i] = cmk(0.0, 0.0);
        if (HOP) {
            int nf[4], nbk[4], par;
            unsigned wrap;
            tiled_neighbours(g, s, nf, nbk, &wrap, &par);
            const FieldOf<double> in(a.in_hop, nullptr, sys, half);
            PairAcc<double> acc;
            pair_zero(acc);
            parity_dir<0, G5HOP>(a, in, s, nf, nbk, wrap, c, sg, acc);
            parity_dir<1, G5HOP>(a, in, s, nf, nbk, wrap, c, sg, acc);
            parity_dir<2, G5HOP>(a, in, s, nf, nbk, wrap, c, sg, acc);
            parity_dir<3, G5HOP>(a, in, s, nf, nbk, wrap, c, sg, acc);
            pair_finish(acc, lower, v);
            const double f = -0.5 * a.hop_sign;
#pragma unroll
            for (int i = 0; i < 6; ++i) v.v[i] = f * v.v[i];
        }
        if (DIAG) {
            Chir<double> d;
            FieldOf<double>(a.in_diag, nullptr, sys, half).chirality(h, c, d);
            if (a.g5_diag && lower) {
#pragma unroll
                for (int i = 0; i < 6; ++i) d.v[i] = -d.v[i];
            }
            double A[36];
            const size_t ca = (size_t)(9 * c) * g.V + s;
#pragma unroll
            for (int k = 0; k < 9; ++k) Unit<double>::load(plane<double>(a.clover, k, g.V), ca, A + 4 * k);
            clover_block_acc(A, lower ? -mu : mu, d.v, v.v);
        }
        if (a.in_add) {
            Chir<double> d;
            FieldOf<double>(a.in_add, nullptr, sys, half).chirality(h, c, d);
#pragma unroll
            for (int i = 0; i < 6; ++i) v.v[i] = v.v[i] + a.add_sign * d.v[i];
        }
        if (INV) {
            const void* inv = a.inv[a.sel[sys]];
            const size_t ia = (size_t)(18 * c) * half + h;
            Chir<double> o;
#pragma unroll
            for (int i = 0; i < 6; ++i) o.v[i] = cmk(0.0, 0.0);
#pragma unroll
            for (int u = 0; u < 18; ++u) {
                double m[4];
                Unit<double>::load(plane<double>(inv, u, half), ia, m);
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int e = 2 * u + k, i = e / 6, j = e % 6;
                    const cplx<double> z = cmk(m[2 * k], m[2 * k + 1]);
                    if (mu < 0)  // the adjoint: the inverse for the opposite twist
                        o.v[j] = cjmad(z, v.v[i], o.v[j]);
                    else
                        o.v[i] = cmad(z, v.v[j], o.v[i]);
                }
            }
            v = o;
        }
        if (a.g5_out && lower) {
#pragma unroll
            for (int i = 0; i < 6; ++i) v.v[i] = -v.v[i];
        }
        if (on) {
            store_chir<double, double>(a.out + (size_t)sys * 6 * half * 4, nullptr, half, h, c, v);
#pragma unroll
            for (int i = 0; i < 6; ++i) n2 += v.v[i].re * v.v[i].re + v.v[i].im * v.v[i].im;
        }
    }
    if (a.partials) {
        n2 = wave_sum(n2);
        if (lane == 0) nrm[w] = n2;
        __syncthreads();
        const int k = threadIdx.x;
        if (k < TILE && (int)blockIdx.y * TILE + k < a.nsys)
            a.partials[((size_t)(blockIdx.y * TILE + k) * blocks + first) * TILE + part] = sum_parts<runs>(nrm + k * runs);
    }
}

// canonical complex128 [nsys][V][4][3] <-> the two compact parity fields
__global__ void __launch_bounds__(kThreads) k_parity_import(Geo g, int nsys, const double* __restrict__ canon,
                                                            double* even, double* odd, unsigned* flag) {
    const long long half = g.V / 2;
    const long long h = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int sys = blockIdx.y;
    if (h >= half || sys >= nsys) return;
    for (int k = 0; k < 2; ++k) {
        const unsigned s = 2u * (unsigned)h + k;
        int c[4];
        site_coords(g, s, c);
        const double2* p = reinterpret_cast<const double2*>(canon) + ((size_t)sys * g.V + lex_site(g, c)) * 12;
        Spinor<double> v;
        bool bad = false;
        for (int i = 0; i < 12; ++i) {
            const double2 t = p[i];
            v.v[i] = cmk(t.x, t.y);
            bad |= !isfinite(t.x) || !isfinite(t.y);
        }
        if (bad) atomicOr(flag, 1u);
        double* dst = ((c[0] + c[1] + c[2] + c[3]) & 1) ? odd : even;
        store_spinor<double, double>(dst + (size_t)sys * 6 * half * 4, nullptr, half, h, v);
    }
}

__global__ void __launch_bounds__(kThreads) k_parity_export(Geo g, int nsys, const double* __restrict__ even,
                                                            const double* __restrict__ odd, double* canon) {
    const long long half = g.V / 2;
    const long long h = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int sys = blockIdx.y;
    if (h >= half || sys >= nsys) return;
    for (int k = 0; k < 2; ++k) {
        const unsigned s = 2u * (unsigned)h + k;
        int c[4];
        site_coords(g, s, c);
        const double* src = ((c[0] + c[1] + c[2] + c[3]) & 1) ? odd : even;
        Spinor<double> v;
        load_spinor<double, double>(src + (size_t)sys * 6 * half * 4, nullptr, half, h, v);
        double2* p = reinterpret_cast<double2*>(canon) + ((size_t)sys * g.V + lex_site(g, c)) * 12;
        for (int i = 0; i < 12; ++i) p[i] = make_double2(v.v[i].re, v.v[i].im);
    }
}

// y = a[sys] x + b[sys] y on compact fields (a, b real, per system)
__global__ void __launch_bounds__(kThreads) k_axpby(const double* __restrict__ x, const double* a, double* y,
                                                    const double* b, long long n_per_sys) {
    const int sys = blockIdx.y;
    const double fa = a[sys], fb = b[sys];
    const double* xs = x + (size_t)sys * n_per_sys;
    double* ys = y + (size_t)sys * n_per_sys;
    for (long long i = (long long)blockIdx.x * kThreads + threadIdx.x; i < n_per_sys;
         i += (long long)gridDim.x * kThreads)
        ys[i] = fa * xs[i] + fb * ys[i];
}

// Sum of n partials of PARTS parts each, in the same order in every workgroup that forms it.
template <int PARTS>
__device__ inline double sum_partials(const double* p, int n, double* lds) {
    double t = 0;
    for (int i = threadIdx.x; i < n; i += kThreads) t += sum_parts<PARTS>(p + (size_t)PARTS * i);
    t = wave_sum(t);
    __syncthreads();  // earlier reads of lds
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = t;
    __syncthreads();
    return (lds[0] + lds[1]) + (lds[2] + lds[3]);
}

// The vector updates of one CG step.  The scalars are formed where they are used, by every workgroup from
// the partial sums that the operator kernels left (deterministic), so that a step is six launches instead of
// fifteen; the state that a step changes (gamma, frozen) is read from one set and written to another.  Frozen
// systems take zero steps.  Bandwidth: 8.9 and 13.5 us for 38 and 63 MB on 16^3x32, in place of 3 axpby, 3 norms
// with their sums and 2 scalar kernels (56 us); a whole solve there went from 31.3 to 23.3 ms.
//   first:  alpha = gamma / <q,q>;  r -= alpha q, partials of <r,r>
//   second: beta = <s,s> / gamma;  x += alpha p;  p = s + beta p;  gamma' = <s,s>;  frozen' once
//           ||r|| <= limit;  <r,r> to rr
template <int PARTS>
__global__ void __launch_bounds__(kThreads) k_cg_first(CgStep a) {
    __shared__ double lds[4];
    const int sys = blockIdx.y;
    const double qq = sum_partials<PARTS>(a.qq + (size_t)sys * a.n_op * PARTS, a.n_op, lds);
    const double al = (a.frozen[sys] != 0 || !(qq > 0)) ? 0.0 : a.gamma[sys] / qq;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.alpha[sys] = al;
    const double2* q = reinterpret_cast<const double2*>(a.q + (size_t)sys * a.n);
    double2* r = reinterpret_cast<double2*>(a.r + (size_t)sys * a.n);
    double n2 = 0;
    for (long long i = (long long)blockIdx.x * kThreads + threadIdx.x; i < a.n / 2; i += (long long)gridDim.x * kThreads) {
        double2 v = r[i];
        const double2 w = q[i];
        v.x -= al * w.x;
        v.y -= al * w.y;
        r[i] = v;
        n2 += v.x * v.x;
        n2 += v.y * v.y;
    }
    n2 = wave_sum(n2);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = n2;
    __syncthreads();
    if (threadIdx.x == 0) a.rr_part[(size_t)sys * gridDim.x + blockIdx.x] = (lds[0] + lds[1]) + (lds[2] + lds[3]);
}

template <int PARTS>
__global__ void __launch_bounds__(kThreads) k_cg_second(CgStep a) {
    __shared__ double lds[4];
    const int sys = blockIdx.y;
    const double ss = sum_partials<PARTS>(a.ss + (size_t)sys * a.n_op * PARTS, a.n_op, lds);
    const bool off = a.frozen[sys] != 0;
    const double gam = a.gamma[sys], al = a.alpha[sys], be = (off || !(gam > 0)) ? 0.0 : ss / gam;
    if (blockIdx.x == 0) {
        const double rr = sum_partials<1>(a.rr_part + (size_t)sys * a.n_rr, a.n_rr, lds);
        if (threadIdx.x == 0) {
            a.gamma_next[sys] = off ? gam : ss;
            a.frozen_next[sys] = (off || sqrt(fmax(0.0, rr)) <= a.limit[sys]) ? 1.0 : 0.0;
            a.rr[sys] = rr;
        }
    }
    if (off) return;
    const double2* s = reinterpret_cast<const double2*>(a.s + (size_t)sys * a.n);
    double2* p = reinterpret_cast<double2*>(a.p + (size_t)sys * a.n);
    double2* x = reinterpret_cast<double2*>(a.x + (size_t)sys * a.n);
    for (long long i = (long long)blockIdx.x * kThreads + threadIdx.x; i < a.n / 2; i += (long long)gridDim.x * kThreads) {
        const double2 sv = s[i];
        double2 pv = p[i], xv = x[i];
        xv.x += al * pv.x;
        xv.y += al * pv.y;
        x[i] = xv;
        pv.x = sv.x + be * pv.x;
        pv.y = sv.y + be * pv.y;
        p[i] = pv;
    }
}

}  // namespace

int parity_parts(int nsys) { return nsys > 2 ? 4 : nsys; }

// One statement for PARTS = 1, 2 or 4 (parity_parts).
#define TM_PARTS_DISPATCH(n, ...)           \
    do {                                    \
        if ((n) == 1) {                     \
            constexpr int PARTS = 1;        \
            __VA_ARGS__;                    \
        } else if ((n) == 2) {              \
            constexpr int PARTS = 2;        \
            __VA_ARGS__;                    \
        } else {                            \
            constexpr int PARTS = 4;        \
            __VA_ARGS__;                    \
        }                                   \
    } while (0)

static int parity_chunks(const Geo& g) { return (int)((g.V / 2 + 127) / 128); }

// At most 2048 (every workgroup of the update kernels adds up the partial sums, up to four per block), a multiple of
// the 8 XCDs, so that a workgroup stays with its XCD's sites; by V alone.
int parity_blocks(const Geo& g) {
    const int n = (parity_chunks(g) + 7) / 8 * 8;
    return n < 2048 ? n : 2048;
}

hipError_t launch_parity_op(const ParityArgs& args, hipStream_t st) {
    ParityArgs a = args;
    a.sys_tile = parity_parts(a.nsys);
    a.chunks = parity_chunks(a.g);
    const dim3 grid((unsigned)(parity_blocks(a.g) * a.sys_tile), (unsigned)((a.nsys + a.sys_tile - 1) / a.sys_tile)),
        blk(kThreads);
    const bool hop = a.in_hop != nullptr, diag = a.in_diag != nullptr, inv = a.do_inv != 0;
#define TM_PARITY_LAUNCH(...) TM_PARTS_DISPATCH(a.sys_tile, hipLaunchKernelGGL((k_parity_op<__VA_ARGS__, PARTS>), grid, blk, 0, st, a))
    if (hop && !diag && inv && a.g5_hop)
        TM_PARITY_LAUNCH(true, false, true, true);
    else if (hop && !diag && inv)
        TM_PARITY_LAUNCH(true, false, true, false);
    else if (hop && diag && !inv && !a.g5_hop)
        TM_PARITY_LAUNCH(true, true, false, false);
    else if (hop && !diag && !inv && !a.g5_hop)
        TM_PARITY_LAUNCH(true, false, false, false);
    else if (!hop && !diag && inv)
        TM_PARITY_LAUNCH(false, false, true, false);
    else
        return hipErrorInvalidValue;
#undef TM_PARITY_LAUNCH
    return hipGetLastError();
}

hipError_t launch_parity_import(const Geo& g, int nsys, const void* canon, double* even, double* odd, unsigned* flag,
                                hipStream_t st) {
    const long long half = g.V / 2;
    hipLaunchKernelGGL(k_parity_import, dim3((unsigned)((half + kThreads - 1) / kThreads), nsys), dim3(kThreads), 0,
                       st, g, nsys, (const double*)canon, even, odd, flag);
    return hipGetLastError();
}

hipError_t launch_parity_export(const Geo& g, int nsys, const double* even, const double* odd, void* canon,
                                hipStream_t st) {
    const long long half = g.V / 2;
    hipLaunchKernelGGL(k_parity_export, dim3((unsigned)((half + kThreads - 1) / kThreads), nsys), dim3(kThreads), 0,
                       st, g, nsys, even, odd, (double*)canon);
    return hipGetLastError();
}

hipError_t launch_axpby(const double* x, const double* a, double* y, const double* b, int nsys, long long n_per_sys,
                        hipStream_t st) {
    const long long nb = (n_per_sys + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(k_axpby, dim3((unsigned)(nb < 4096 ? nb : 4096), nsys), dim3(kThreads), 0, st, x, a, y, b,
                       n_per_sys);
    return hipGetLastError();
}

int cg_blocks(long long n) {
    const long long nb = (n / 2 + kThreads - 1) / kThreads;
    return (int)(nb < 1024 ? nb : 1024);
}

hipError_t launch_cg_first(const CgStep& a, int nsys, hipStream_t st) {
    TM_PARTS_DISPATCH(a.parts, hipLaunchKernelGGL(k_cg_first<PARTS>, dim3((unsigned)cg_blocks(a.n), nsys), dim3(kThreads), 0, st, a));
    return hipGetLastError();
}

hipError_t launch_cg_second(const CgStep& a, int nsys, hipStream_t st) {
    TM_PARTS_DISPATCH(a.parts, hipLaunchKernelGGL(k_cg_second<PARTS>, dim3((unsigned)cg_blocks(a.n), nsys), dim3(kThreads), 0, st, a));
    return hipGetLastError();
}

}  // namespace tmsap
