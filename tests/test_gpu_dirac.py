"""GPU operator parity: tm_dirac_apply (HIP) against the FP64 CPU oracle.

Each application is checked norm-wise and per site against the error model of
gpu_util (f64 1e-13, f32 2e-6, f16 2e-3, bf16 1.5e-2).
"""
import numpy as np
import pytest

import oracle
import paper_1610_02370_amd as tm
from paper_1610_02370_amd import synth

from gpu_util import TOL as ERR_TOL
from gpu_util import announce, check_close, dev, host, rel_err

pytestmark = pytest.mark.gpu

TOL = ERR_TOL["dirac"]

CASES = [
    # dims, eps, kappa, mus, csw, antiperiodic; dims chosen so tiles are mixed
    # (4 and 2 per axis) and the last 256-thread group is partly filled
    ((8, 6, 4, 10), 0.5, 0.1632, [0.003], 1.5, False),
    ((4, 4, 4, 4), 0.3, 0.16, [0.01, -0.01], 0.0, True),
    ((6, 4, 8, 4), 0.6, 0.1373, [0.0009, -0.0009, 0.0009], 1.5, False),
    # 4^4 tiles (the tiled FP32 kernel): 2, 3, 1, 2 blocks per axis, so one axis has an odd
    # count and along y the block is its own neighbour
    ((8, 12, 4, 8), 0.55, 0.15, [0.004, -0.004, 0.01], 1.2, True),
]


@pytest.fixture(scope="module")
def fields():
    out = []
    for k, (dims, eps, kappa, mus, csw, ap) in enumerate(CASES):
        U = synth.gauge_field(dims, eps, seed=20 + k)
        psi = synth.gaussian_spinor(dims, len(mus), seed=120 + k)
        op = oracle.Operator(dims, U, oracle.kappa_to_m(kappa), 0.0, csw, antiperiodic_t=ap)
        ref = np.stack([op.with_mu(m).apply(psi[i]).reshape(-1, 4, 3) for i, m in enumerate(mus)])
        out.append((U, psi, ref))
    return out


@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_dirac_matches_oracle(fields, case, prec):
    dims, eps, kappa, mus, csw, ap = CASES[case]
    U, psi, ref = fields[case]
    announce(f"dirac parity case={case} dims={dims} prec={prec}")
    out = tm.tm_dirac_apply(dims, dev(U), dev(psi), kappa, mus, csw, storage=prec, antiperiodic_t=ap)
    got = host(out)
    for i in range(len(mus)):
        check_close(got[i], ref[i], "dirac", prec, f"case {case} {dims} system {i}")


def test_dirac_internal_io_roundtrip(fields):
    import torch

    dims, eps, kappa, mus, csw, ap = CASES[0]
    U, psi, ref = fields[0]
    announce("dirac internal-io roundtrip")
    for prec in ("f64", "f32"):
        nbytes = tm.tm_spinor_bytes(dims, len(mus), prec)
        a = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        b = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        tm.tm_spinor_import(dims, dev(psi), a, storage=prec)
        tm.tm_dirac_apply(dims, dev(U), a, kappa, mus, csw, b, storage=prec, io="internal")
        out = torch.empty_like(dev(psi))
        tm.tm_spinor_export(dims, b, out, storage=prec)
        assert rel_err(host(out)[0], ref[0]) < TOL[prec]
        back = torch.empty_like(out)
        tm.tm_spinor_export(dims, a, back, storage=prec)
        if prec == "f64":
            assert np.array_equal(host(back), psi)


def test_fp16_scale_subnormal_and_zero_sites():
    # FP16 storage scales each site by a power of two: a site whose largest component is an FP32
    # subnormal (about 1e-40, where a reciprocal scale would overflow) and an all-zero site must
    # come back finite, the first within FP16 rounding of its own size, the second exactly zero
    import torch

    dims = (4, 4, 4, 4)
    rng = np.random.default_rng(11)
    psi = rng.normal(size=(1, 256, 4, 3)) + 1j * rng.normal(size=(1, 256, 4, 3))
    psi[0, 1] *= 1e-40          # FP32 subnormal band
    psi[0, 2] *= 3e-39          # just below the smallest normal FP32 number
    psi[0, 3] = 0.0             # zero site
    psi[0, 4] *= 1e30           # large site: FP16 alone would overflow
    announce("fp16 storage: subnormal, zero and large sites")
    nbytes = tm.tm_spinor_bytes(dims, 1, "f16")
    a = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    tm.tm_spinor_import(dims, dev(psi), a, storage="f16")
    back = host(tm.tm_spinor_export(dims, a, dev(np.zeros_like(psi)), storage="f16"))
    assert np.isfinite(back).all()
    assert np.array_equal(back[0, 3], psi[0, 3])
    for s in range(256):
        if s == 3:
            continue
        m = np.abs(np.concatenate([psi[0, s].real.ravel(), psi[0, s].imag.ravel()])).max()
        err = np.abs(np.concatenate([(back[0, s] - psi[0, s]).real.ravel(), (back[0, s] - psi[0, s]).imag.ravel()]))
        # one FP16 rounding (2^-11 of the power-of-two scale, which is < 2 m), plus the FP32 subnormal
        # spacing 2^-149 for the tiny sites
        assert err.max() <= 2.0 ** -11 * 2 * m + 2.0 ** -149, (s, err.max(), m)


def test_dirac_gamma5_hermiticity_on_gpu(fields):
    # <phi, D(mu) psi> = <Gamma5 D(-mu) Gamma5 phi, psi>, both sides from the GPU
    dims, eps, kappa, mus, csw, ap = CASES[2]
    U, psi, _ = fields[2]
    announce("dirac gamma5-hermiticity on GPU")
    rng = np.random.default_rng(7)
    phi = rng.normal(size=psi[:1].shape) + 1j * rng.normal(size=psi[:1].shape)
    g5 = np.array([1, 1, -1, -1])[None, None, :, None]
    Dpsi = host(tm.tm_dirac_apply(dims, dev(U), dev(psi[:1]), kappa, [0.2], csw))
    Dphi = host(tm.tm_dirac_apply(dims, dev(U), dev(g5 * phi), kappa, [-0.2], csw))
    lhs = np.vdot(phi.ravel(), Dpsi.ravel())
    rhs = np.vdot((g5 * Dphi).ravel(), psi[:1].ravel())
    assert abs(lhs - rhs) < 1e-12 * abs(lhs)


def test_dirac_error_paths(fields):
    dims, eps, kappa, mus, csw, ap = CASES[0]
    U, psi, _ = fields[0]
    announce("dirac error paths")
    with pytest.raises(tm.TMError) as e:
        tm.tm_dirac_apply(dims, dev(1.1 * U), dev(psi), kappa, mus, csw)
    assert e.value.code == -8
    bad = U.copy()
    bad[3, 1, 0, 0] = np.nan
    with pytest.raises(tm.TMError) as e:
        tm.tm_dirac_apply(dims, dev(bad), dev(psi), kappa, mus, csw)
    assert e.value.code == -7
    with pytest.raises(tm.TMError) as e:
        tm.tm_dirac_apply(dims, dev(U), dev(psi), kappa, mus, csw, layout_block=(3, 3, 4, 5))
    assert e.value.code == -2
    t = dev(psi)
    with pytest.raises(tm.TMError) as e:
        tm.tm_dirac_apply(dims, dev(U), t, kappa, mus, csw, t)
    assert e.value.code == -1


def test_gauge_tag_rebuilds_the_same_buffer_in_place(fields):
    # a new tag for the same U buffer after its contents changed: the library rebuilds that
    # buffer's cached copy (in place) and every later call with the new tag uses the new field
    dims, eps, kappa, mus, csw, ap = CASES[3]
    U1, psi, ref1 = fields[3]
    U2 = synth.gauge_field(dims, eps, seed=99)
    op2 = oracle.Operator(dims, U2, oracle.kappa_to_m(kappa), 0.0, csw, antiperiodic_t=ap)
    ref2 = np.stack([op2.with_mu(m).apply(psi[i]).reshape(-1, 4, 3) for i, m in enumerate(mus)])
    announce("gauge tag: same buffer, new contents, new tag")
    Ud = dev(U1)
    for prec in ("f32", "f64"):
        got = host(tm.tm_dirac_apply(dims, Ud, dev(psi), kappa, mus, csw, storage=prec, antiperiodic_t=ap,
                                     gauge_tag=5))
        for i in range(len(mus)):
            check_close(got[i], ref1[i], "dirac", prec, f"tag 5 field 1 system {i}")
    Ud.copy_(dev(U2))
    for rep in range(2):  # the first call rebuilds, the second reuses the rebuilt copy
        for prec in ("f32", "f64"):
            got = host(tm.tm_dirac_apply(dims, Ud, dev(psi), kappa, mus, csw, storage=prec, antiperiodic_t=ap,
                                         gauge_tag=6))
            for i in range(len(mus)):
                check_close(got[i], ref2[i], "dirac", prec, f"tag 6 field 2 call {rep} system {i}")
    tm.tm_gauge_release(Ud)


@pytest.mark.parametrize("prec", ["f32", "f16"])
def test_dirac_64_systems_match_single_calls(prec):
    # the tiled FP32 operator loops over every system of the call inside each workgroup; the
    # largest batch the ABI allows gives, system by system, the bits of one-system calls
    dims = (8, 8, 8, 8)
    U = synth.gauge_field(dims, 0.5, seed=61)
    mus = [0.002 * (k - 32) for k in range(64)]
    psi = synth.gaussian_spinor(dims, len(mus), seed=161)
    announce(f"dirac 64 systems vs single calls, {prec}")
    Ud = dev(U)
    allsys = host(tm.tm_dirac_apply(dims, Ud, dev(psi), 0.15, mus, 1.2, storage=prec))
    for k in (0, 1, 31, 32, 63):
        one = host(tm.tm_dirac_apply(dims, Ud, dev(psi[k:k + 1]), 0.15, [mus[k]], 1.2, storage=prec))
        assert np.array_equal(allsys[k], one[0]), k
    op = oracle.Operator(dims, U, oracle.kappa_to_m(0.15), 0.0, 1.2)
    for k in (0, 63):
        ref = op.with_mu(mus[k]).apply(psi[k]).reshape(-1, 4, 3)
        check_close(allsys[k], ref, "dirac", prec, f"64 systems, system {k}")


@pytest.mark.parametrize("dims,csw", [((4, 4, 4, 4), 1.5), ((1, 3, 2, 5), 1.2), ((5, 3, 7, 9), 0.7), ((2, 8, 4, 12), 0.0)])
def test_gauge_build_with_and_without_staged_links(dims, csw):
    # the clover term from time slices staged as a structure of arrays, against the oracle, on lattices whose
    # slices are not multiples of a workgroup's 64 sites, extents of 1 and 2 wrap onto themselves, or the term is zero
    U, psi = synth.gauge_field(dims, 0.6, seed=81), synth.gaussian_spinor(dims, 1, seed=181)
    op = oracle.Operator(dims, U, oracle.kappa_to_m(0.14), 0.1, csw)
    ref = op.apply(psi[0]).reshape(psi[0].shape)
    announce(f"gauge build dims={dims} csw={csw}")
    for tag in (0, 7):
        got = host(tm.tm_dirac_apply(dims, dev(U), dev(psi), 0.14, [0.1], csw, gauge_tag=tag))
        check_close(got[0], ref, "dirac", "f64", f"gauge build {dims} c_sw {csw} tag {tag}")


def test_gauge_build_in_chunks_of_slices():
    # more slices than the staging workspace holds at once: rows of tiles with one slice on either side, the first and
    # last of them wrapping around the lattice
    dims = (48, 32, 32, 32)
    U, psi = synth.gauge_field(dims, 0.6, seed=82), synth.gaussian_spinor(dims, 1, seed=182)
    tm.tm_finalize()  # no workspace from an earlier call: 256 MiB hold 14 of the 48 slices
    announce("gauge build in chunks 32^3x48")
    got = host(tm.tm_dirac_apply(dims, dev(U), dev(psi), 0.1373, [0.001], 1.5))[0].reshape(dims + (4, 3))
    for t in (0, 1, 11, 12, 23, 47):  # windows of slices t - 2 .. t + 2 hold everything that slice t needs
        w = [(t + k) % dims[0] for k in range(-2, 3)]
        Uw = U.reshape(dims + (4, 3, 3))[w].reshape(-1, 4, 3, 3)
        op = oracle.Operator((5,) + dims[1:], Uw, oracle.kappa_to_m(0.1373), 0.001, 1.5)
        ref = op.apply(psi[0].reshape(dims + (4, 3))[w].reshape(-1, 4, 3)).reshape((5,) + dims[1:] + (4, 3))[2]
        check_close(got[t], ref, "dirac", "f64", f"slice {t}")


@pytest.mark.parametrize("dims,nsys", [((3, 5, 7, 9), 1), ((3, 5, 7, 9), 2), ((6, 10, 7, 9), 9), ((8, 8, 16, 20), 5), ((4, 4, 4, 4), 2)])
def test_canonical_application_matches_staged_one(dims, nsys):
    # FP64 on the caller's canonical buffers (directions split over wavefronts up to 32768 sites times systems, one
    # wavefront per system and site above), against internal buffers and, with overlapping buffers, the staged path
    import torch

    mus = [0.1 * (k - 1) for k in range(nsys)]
    U, psi = synth.gauge_field(dims, 0.6, seed=91), synth.gaussian_spinor(dims, nsys, seed=191)
    kw = dict(antiperiodic_t=True, theta=(0.2, 0.3, -0.9, 0.5), mu_shift=(0.03, -0.02))
    op = oracle.Operator(dims, U, oracle.kappa_to_m(0.14), 0.0, 1.2, **kw)
    announce(f"canonical application dims={dims} nsys={nsys}")
    Ud, p = dev(U), dev(psi)
    got = host(tm.tm_dirac_apply(dims, Ud, p, 0.14, mus, 1.2, **kw))
    for k in range(nsys):
        check_close(got[k], op.with_mu(mus[k]).apply(psi[k]), "dirac", "f64", f"canonical {dims} system {k}")
    n = tm.tm_spinor_bytes(dims, nsys, "f64")
    a, b = (torch.zeros(n, dtype=torch.uint8, device="cuda") for _ in range(2))
    tm.tm_spinor_import(dims, p, a, storage="f64")
    tm.tm_dirac_apply(dims, Ud, a, 0.14, mus, 1.2, b, io="internal", **kw)
    inner = host(tm.tm_spinor_export(dims, b, torch.empty_like(p), storage="f64"))
    assert rel_err(inner, got) < 1e-13
    both = torch.empty((p.numel() + 12,), dtype=torch.complex128, device="cuda")  # out one site behind psi
    both[:p.numel()] = p.reshape(-1)
    out = both[12:].view(p.shape)
    tm.tm_dirac_apply(dims, Ud, both[:p.numel()].view(p.shape), 0.14, mus, 1.2, out, **kw)
    assert rel_err(host(out), got) < 1e-13


# Boxes of the clover build: steps of 4 and of 3, boxes cut off by the lattice's end, one and two slices.
@pytest.mark.parametrize("dims", [(2, 6, 10, 7), (4, 9, 5, 3), (3, 11, 4, 6), (6, 2, 1, 14)])
def test_clover_build_boxes(dims):
    U, psi = synth.gauge_field(dims, 0.6, seed=83), synth.gaussian_spinor(dims, 1, seed=183)
    ref = oracle.Operator(dims, U, oracle.kappa_to_m(0.14), 0.1, 1.3).apply(psi[0]).reshape(psi[0].shape)
    announce(f"clover boxes dims={dims}")
    got = host(tm.tm_dirac_apply(dims, dev(U), dev(psi), 0.14, [0.1], 1.3))
    check_close(got[0], ref, "dirac", "f64", f"clover boxes {dims}")


# 20480 (4^4 tiles) and 20160 sites: one system alone has its directions split over wavefronts, several together have
# not, and in internal buffers on 4^4 tiles, or on other tiles where these fill the device (23^2x19^2, the last workgroup
# partly filled), they take the kernel with one lane per site.  One order of sums for all.
@pytest.mark.parametrize("dims", [(8, 8, 16, 20), (7, 9, 16, 20), (23, 19, 19, 23)])
def test_system_of_a_batch_is_bit_identical_to_it_alone(dims):
    import torch

    mus = [0.1, -0.02, 0.3]
    U, psi = dev(synth.gauge_field(dims, 0.6, seed=93)), dev(synth.gaussian_spinor(dims, len(mus), seed=193))
    kw = dict(antiperiodic_t=True, theta=(0.2, 0.3, -0.9, 0.5), mu_shift=(0.03, -0.02), gauge_tag=9)
    announce(f"batch and single applications dims={dims}")

    def internal(p, m):
        n = tm.tm_spinor_bytes(dims, len(m), "f64")
        a, b = (torch.zeros(n // 8, dtype=torch.float64, device="cuda") for _ in range(2))
        tm.tm_spinor_import(dims, p, a, storage="f64")
        tm.tm_dirac_apply(dims, U, a, 0.14, m, 1.2, b, io="internal", **kw)
        return tm.tm_spinor_export(dims, b, torch.empty_like(p), storage="f64")

    batch = tm.tm_dirac_apply(dims, U, psi, 0.14, mus, 1.2, **kw)
    assert torch.equal(internal(psi, mus), batch)
    for k, m in enumerate(mus):
        p = psi[k:k + 1].contiguous()
        assert torch.equal(tm.tm_dirac_apply(dims, U, p, 0.14, [m], 1.2, **kw), batch[k:k + 1])
        assert torch.equal(internal(p, [m]), batch[k:k + 1])


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
def test_flexible_steps_of_a_batch_are_bit_identical_to_single_ones(storage):
    # the FP64 operator on vectors of the smoother's precision, split over wavefronts for one system and not for two
    import torch

    dims, mus = (8, 8, 16, 24), [0.001, -0.002]
    U, b = dev(synth.gauge_field(dims, 0.5, seed=94)), dev(synth.gaussian_spinor(dims, 2, seed=194))
    announce(f"flexible steps, batch and single, {storage}")

    def solve(k0, k1):
        x = torch.zeros_like(b[k0:k1])
        tm.tm_fgmres_solve(dims, U, b[k0:k1].contiguous(), x, 0.1373, mus[k0:k1], 1.5, 1e-12, storage=storage,
                           form="flexible", restart=10, n_cycles=2, mr_iters=3, block_dims=(4, 4, 4, 4), x_in=False,
                           max_iters=6, gauge_tag=11)
        return x

    both = solve(0, 2)
    for k in range(2):
        assert torch.equal(solve(k, k + 1), both[k:k + 1])


def test_fp32_application_of_one_round_of_tiles():
    # 512 tiles, as many as run at once, with seven systems in each workgroup: the operator that reads the upper halo
    # where it is staged; every system alone takes the other one.  The same sums in both.
    import torch

    dims, mus = (32, 16, 16, 16), [0.01 * (k - 3) for k in range(7)]
    U, psi = dev(synth.gauge_field(dims, 0.6, seed=95)), dev(synth.gaussian_spinor(dims, len(mus), seed=195))
    announce("FP32 application, 512 tiles, seven systems")
    kw = dict(storage="f32", theta=(0.2, 0.3, -0.9, 0.5), gauge_tag=13)
    batch = tm.tm_dirac_apply(dims, U, psi, 0.14, mus, 1.2, **kw)
    for k, m in enumerate(mus):
        assert torch.equal(tm.tm_dirac_apply(dims, U, psi[k:k + 1].contiguous(), 0.14, [m], 1.2, **kw), batch[k:k + 1])


def test_defect_correction_steps_of_a_batch_are_bit_identical_to_single_ones():
    # six systems on 512 tiles of a colour: D z on one colour's tiles from the same operator, two ways as above
    import torch

    dims, mus = (32, 32, 16, 16), [0.001 * (k - 2) for k in range(6)]
    U, b = dev(synth.gauge_field(dims, 0.5, seed=96)), dev(synth.gaussian_spinor(dims, len(mus), seed=196))
    announce("defect-correction steps, batch and single")

    def solve(k0, k1):
        x = torch.zeros_like(b[k0:k1])
        tm.tm_fgmres_solve(dims, U, b[k0:k1].contiguous(), x, 0.1373, mus[k0:k1], 1.5, 1e-12, storage="f32",
                           form="defect_correction", restart=8, n_cycles=2, mr_iters=3, block_dims=(4, 4, 4, 4),
                           x_in=False, max_iters=4, gauge_tag=15)
        return x

    batch = solve(0, len(mus))
    for k in range(len(mus)):
        assert torch.equal(solve(k, k + 1), batch[k:k + 1])


# Many systems on few tiles: several stay in each workgroup of the generic kernel (15 workgroups, 40 systems) and of the
# one for 4^4 tiles (32 tiles, 64 systems), whose loops over systems then run more than once.
@pytest.mark.parametrize("prec", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("dims,nsys", [((6, 10, 7, 9), 40), ((8, 8, 8, 16), 64)])
def test_system_loop_of_the_application(dims, nsys, prec):
    mus = [0.002 * (k - 20) for k in range(nsys)]
    U, psi = synth.gauge_field(dims, 0.5, seed=98), synth.gaussian_spinor(dims, nsys, seed=198)
    announce(f"application of {nsys} systems dims={dims} prec={prec}")
    Ud = dev(U)
    got = host(tm.tm_dirac_apply(dims, Ud, dev(psi), 0.15, mus, 1.2, storage=prec, gauge_tag=17))
    op = oracle.Operator(dims, U, oracle.kappa_to_m(0.15), 0.0, 1.2)
    for k in (0, 1, 2, 3, nsys // 2, nsys - 2, nsys - 1):
        one = tm.tm_dirac_apply(dims, Ud, dev(psi[k:k + 1]), 0.15, [mus[k]], 1.2, storage=prec, gauge_tag=17)
        assert np.array_equal(got[k], host(one)[0]), k
    for k in (2, nsys - 1):
        check_close(got[k], op.with_mu(mus[k]).apply(psi[k]).reshape(-1, 4, 3), "dirac", prec, f"{nsys} systems {dims} {k}")
