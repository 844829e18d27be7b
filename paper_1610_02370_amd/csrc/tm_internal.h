// Host-side declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "tm_device.h"

namespace tmsap {

enum Prec { P_F64 = 0, P_F32 = 1, P_F16 = 2, P_BF16 = 3 };

constexpr int kMaxSys = 64;

inline int unit_bytes(Prec p) { return p == P_F64 ? 32 : (p == P_F32 ? 16 : 8); }
inline bool prec_has_scale(Prec p) { return p == P_F16; }

// Internal spinor field: data [nsys][6 units][V], FP16 scales [nsys][V].
struct SpinorBuf {
    void* data = nullptr;
    float* scale = nullptr;
    Prec prec = P_F64;
    int nsys = 0;
};

// Bytes of the data part / scale part of an internal spinor field.
inline size_t spinor_data_bytes(long long V, int nsys, Prec p) { return (size_t)nsys * 6 * V * unit_bytes(p); }
inline size_t spinor_scale_bytes(long long V, int nsys, Prec p) {
    return prec_has_scale(p) ? (size_t)nsys * V * sizeof(float) : 0;
}
// Systems per workgroup of a launch over `blocks` tiles and nsys systems when `slots` workgroups fit
// the device at once.  A workgroup loads its tile's links and clover once (`load`, in units of one
// system's work) and then takes its systems in turn, so all systems in one workgroup is best as long
// as the tiles fill the device; with fewer tiles than slots most of the chip idles while each
// workgroup runs through every system.  The split with the least ceil(workgroups / slots) x
// (systems + load) is taken, unless a coarser one is within 10 % of it (24^3x32 with 2 FP64 systems,
// estimated 5 % better, ran 6 % worse).  Results do not depend on the split.  Measured at 16^4 with 12
// FP32 systems (128 blocks of a colour, 512 slots): the half-sweep 230 us unsplit, the whole
// defect-correction solve 31.1 -> 13.4 ms with the split; a 6x10x7x9 FP64 application of 3 systems
// 44 -> 27 us.  At 48^3x96 (20736 blocks) no split is taken.
//
// fill_only (the operator kernels, bound by memory): no split once the tiles fill the slots.  Their last,
// partly filled wave of workgroups runs faster than a full one, so splitting to even it out lost 10 %
// (16^3x36, 2 systems: FP64 86 -> 97 us, FP32 41 -> 45).
inline int pick_sys_tile(long long blocks, int nsys, int slots, double load, bool fill_only) {
    if (fill_only && blocks >= slots) return nsys;
    int best = nsys;
    double best_cost = 0;
    for (int groups = 1; groups <= nsys; ++groups) {
        const int tile = (nsys + groups - 1) / groups;
        const long long wg = blocks * ((nsys + tile - 1) / tile);
        const double cost = (double)((wg + slots - 1) / slots) * (tile + load);
        if (groups == 1 || cost < 0.9 * best_cost) {
            best = tile;
            best_cost = cost;
        }
    }
    return best;
}
constexpr int kCUs = 256;  // compute units of the MI355X

// Systems per workgroup of the half-sweeps with one thread per site (tm_sap.hip), nt threads per block.  Workgroups
// per CU: FP32 on up to 256 sites two (LDS of k_sap_half_v2, registers of k_sap_half_44), FP64 there one wavefront
// per SIMD, one of the others.  The block's links and clover cost about 0.15 of one system's residual and MR
// steps, 0.4 in FP32 on more than 256 sites.  With one FP64 workgroup per CU and 0.15 throughout, systems were
// split where the blocks fill the device: 6 systems on 864 blocks of a colour, FP64 4^3x2 2575 us unsplit and 2807
// split, BF16 8x4^3 19.3 and 20.6 ms.
inline int sap_sys_tile(long long blocks, int nsys, int nt, bool fp64, bool eo) {
    const int per_cu = eo || nt > 256 ? 1 : fp64 ? 256 / nt : 2;
    return pick_sys_tile(blocks, nsys, per_cu * kCUs, nt > 256 && !fp64 && !eo ? 0.4 : 0.15, false);
}

inline size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

// Gauge data on the device at one precision: links [4][3 units][V] and the
// packed clover [18 units][V] holding (m+4) + clover.
// Site-diagonal inverses for even-odd solves, one set per (|mu|, parity):
// [36 units][V/2] at the clover precision, entry h for the site of that
// parity in the pair (2h, 2h+1) (tile x-extent even); units 0..17 hold
// (A_up + i|mu|)^-1, units 18..35 hold (A_dn - i|mu|)^-1, each 6x6 row-major
// as (re, im) pairs.
constexpr int kMaxEoMu = 8;
struct EoCache {
    int n = 0;
    double absmu[kMaxEoMu] = {};
    int parity[kMaxEoMu] = {};
    void* inv[kMaxEoMu] = {};
    void release();
    ~EoCache() { release(); }
};

struct GaugeDev {
    void* links = nullptr;
    void* clover = nullptr;
    Prec link_prec = P_F64;
    Prec clover_prec = P_F64;
    EoCache* eo = nullptr;  // owned by the cache entry that holds this
};

struct DiracArgs {
    Geo g;
    const void* links;
    const void* clover;
    const void* in;
    const float* in_scale;
    void* out;
    float* out_scale;
    int nsys;
    int sys_tile = 0;    // systems per workgroup (gridDim.y = ceil(nsys / sys_tile)), set by the launcher
    int colour = -1;     // -1: every 4^4 tile; 0 / 1: the blocks of that colour only (tiled operator)
    double mu[kMaxSys];
};

struct SapArgs {
    Geo g;               // tile = Schwarz block
    const void* links;
    const void* clover;
    const void* b;
    const float* b_scale;
    void* x;
    float* x_scale;
    int nsys;            // systems in the buffers
    int sys_tile;        // systems per workgroup (gridDim.y = ceil(nsys / sys_tile)); 0: the launcher's choice
    int colour;
    int mr_iters;
    int own_zero;        // 1: x is zero on this colour's blocks (skip reading it)
    int halo_zero;       // 1: x is zero on the other colour's blocks too (then r = b)
    int eo;              // 1: even-odd preconditioned block solves
    void* w_out = nullptr;  // set (4^4 FP32 kernel, FP32 storage): D x on the swept blocks, written as
                            // b minus the final block residual, [nsys] fields like x
    unsigned long long eo_adj;            // bit k: system k uses the adjoint inverses (mu_k < 0)
    const void* eo_inv[kMaxEoMu];         // inverse sets by |mu|
    unsigned char eo_sel[kMaxSys];        // system -> inverse set
    double mu[kMaxSys];
};

// One step of the even-odd reduced operator on compact parity fields
// [nsys][6 units][V/2] (FP64): out_p = (D_pp^-1)? [hop_sign * H in_hop +
// D_pp in_diag + add_sign * in_add] with H = -1/2 sum of the hops between
// the parities; null inputs are skipped; the Gamma5 flags multiply the hop
// input, the diagonal input and the output (Dhat^+ = Gamma5 Dhat(-mu) Gamma5).
struct ParityArgs {
    Geo g;
    const void* links;   // FP64 [4][3 units][V]
    const void* clover;  // FP64 [18 units][V]
    const void* inv[kMaxEoMu];  // site inverse sets of parity p
    unsigned char sel[kMaxSys];
    int p;
    const double* in_hop;
    double hop_sign;
    const double* in_diag;
    const double* in_add;
    double add_sign;
    int do_inv;
    int g5_hop, g5_diag, g5_out;
    double mu_sign;
    double* out;
    int nsys;
    int sys_tile, chunks;  // systems per workgroup and chunks of 128 sites, set by the launcher
    double* partials;    // parts of ||out||^2 ([nsys][parity_blocks][parity_parts]), or null
    double mu[kMaxSys];
};

// One step's vector updates (k_cg_first, k_cg_second): vectors [nsys][n], scalars [nsys], partial sums
// [nsys][their number].
struct CgStep {
    long long n;
    const double *q, *s;
    double *r, *p, *x;
    const double *qq, *ss;
    int n_op, parts, n_rr;  // parity_blocks and parity_parts (qq, ss), cg_blocks (rr_part)
    double* rr_part;
    const double *gamma, *frozen, *limit;
    double *alpha, *gamma_next, *frozen_next, *rr;
};

// ---- even-odd reduced operator and CG (tm_cg.hip)
hipError_t launch_parity_op(const ParityArgs& a, hipStream_t st);
hipError_t launch_parity_import(const Geo& g, int nsys, const void* canon, double* even, double* odd, unsigned* flag,
                                hipStream_t st);
hipError_t launch_parity_export(const Geo& g, int nsys, const double* even, const double* odd, void* canon,
                                hipStream_t st);
// y = a[sys] x + b[sys] y over n_per_sys doubles per system
hipError_t launch_axpby(const double* x, const double* a, double* y, const double* b, int nsys, long long n_per_sys,
                        hipStream_t st);
int parity_blocks(const Geo& g);            // partial sums per system of launch_parity_op ...
int parity_parts(int nsys);                 // ... and their parts
int cg_blocks(long long n);                 // the same of launch_cg_first
hipError_t launch_cg_first(const CgStep& a, int nsys, hipStream_t st);
hipError_t launch_cg_second(const CgStep& a, int nsys, hipStream_t st);

// ---- layout kernels (tm_layout.hip)
// Internal links from the canonical ones, with the SU(3) check.
hipError_t launch_link_ingest(const Geo& g, Prec G, const void* Ucanon, void* links, unsigned* stats, hipStream_t st);
// The same and the clover term (FP64 arithmetic on the canonical links).  `stage` (stage_bytes, may be none)
// holds time slices of the links as a structure of arrays while the clover is built from them; without
// room for a row of tiles and its neighbours the clover reads the canonical array.
hipError_t launch_gauge_build(const Geo& g, Prec G, Prec C, const void* Ucanon, double m4, double csw, void* links,
                              void* clover, unsigned* stats, void* stage, size_t stage_bytes, hipStream_t st);
size_t gauge_stage_bytes(const Geo& g, int slices);
// FP32 clover [18][V] units from the FP64 one (FP64 [18][V] double4 units) of the same geometry.
hipError_t launch_clover_to_f32(const Geo& g, const void* clover64, void* clover32, hipStream_t st);
hipError_t launch_spinor_import(const Geo& g, const SpinorBuf& dst, const void* canon, unsigned* flag,
                                hipStream_t st);
hipError_t launch_spinor_export(const Geo& g, const SpinorBuf& src, void* canon, hipStream_t st);
hipError_t launch_spinor_convert(const Geo& g, const SpinorBuf& src, const SpinorBuf& dst, hipStream_t st);
// (A_up + i absmu)^-1 and (A_dn - i absmu)^-1 at every site of one parity, from the packed clover (FP64
// arithmetic)
hipError_t launch_eo_inverse(const Geo& g, Prec C, const void* clover, double absmu, int parity, void* inv,
                             hipStream_t st);
inline size_t eo_inverse_bytes(const Geo& g, Prec C) { return (size_t)36 * (g.V / 2) * unit_bytes(C); }

// ---- operator (tm_dirac.hip)
hipError_t launch_dirac(const DiracArgs& a, Prec in_p, Prec out_p, Prec link_p, Prec clover_p, Prec compute,
                        hipStream_t st);

// The FP64 operator on canonical complex128 fields (a.in, a.out [nsys][V][4][3], not overlapping).
hipError_t launch_dirac_canonical(const DiracArgs& a, hipStream_t st);

// ---- smoother (tm_sap.hip)
// The operator on 4^4 tiles with FP32 arithmetic (tm_sap.hip); hipErrorNotSupported for other
// tiles or precision combinations, which launch_dirac then runs in its generic kernel.
hipError_t launch_dirac_44(const DiracArgs& a, Prec in_p, Prec out_p, Prec link_p, Prec clover_p,
                           hipStream_t st);
hipError_t launch_sap_half(const SapArgs& a, Prec spinor_p, Prec link_p, Prec clover_p, Prec compute,
                           hipStream_t st);
// Half-sweeps with two lanes per site (tm_sap_pair.hip): FP64, and even-odd block solves at every
// precision; hipErrorNotSupported for other blocks than 4^4 and for plain FP32 solves.
hipError_t launch_sap_pair(const SapArgs& a, Prec spinor_p, Prec link_p, Prec clover_p, hipStream_t st);
bool sap_supported(Prec spinor_p, Prec link_p, Prec clover_p, Prec compute);
// True when a half-sweep with these storage/link/clover precisions runs the 4^4 FP32 kernel with
// FP32 storage, whose w_out output is then available.
bool sap_fills_w(const Geo& g, Prec sp, Prec lp, Prec cp, bool eo);
size_t sap_lds_bytes(int Vb, Prec compute);

}  // namespace tmsap
