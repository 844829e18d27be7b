"""GPU smoother parity: tm_sap_smooth (HIP) against the FP64 CPU oracle's SAP.

Both sides run the same red-black sweeps (colour 0 first) with MR block solves
on the same seeded inputs and initial guess.  Each result is checked norm-wise
and per site against the error model of gpu_util (f64 1e-13, f32 2e-6,
f16 2e-3, bf16 1.5e-2).
"""
import numpy as np
import pytest

import oracle
import paper_1610_02370_amd as tm
from paper_1610_02370_amd import synth

from gpu_util import TOL as ERR_TOL
from gpu_util import announce, check_close, dev, host, rel_err

pytestmark = pytest.mark.gpu

TOL = ERR_TOL["sap"]

CASES = [
    # dims, block, eps, kappa, mus, csw, cycles, mr, antiperiodic
    ((4, 4, 4, 4), (2, 2, 2, 2), 0.3, 0.16, [0.01], 0.0, 3, 4, False),          # 16-site blocks
    ((8, 8, 8, 8), (4, 4, 4, 4), 0.5, 0.1632, [0.003, -0.003], 1.5, 2, 4, True),  # 256-site blocks
    ((4, 12, 4, 4), (2, 6, 2, 2), 0.6, 0.1394, [0.001], 1.5, 2, 3, False),      # 96 sites: idle lanes
    ((8, 4, 8, 8), (4, 2, 4, 4), 0.6, 0.1373, [0.0009], 1.5, 1, 4, False),      # 128 sites
    ((8, 8, 4, 16), (4, 4, 2, 8), 0.6, 0.1373, [0.0009], 1.5, 1, 2, False),     # 256 sites, long x
    ((8, 8, 8, 16), (4, 4, 4, 8), 0.5, 0.1373, [0.0009], 1.5, 1, 2, False),     # 512 sites: large groups
    ((16, 16, 16, 16), (4, 4, 4, 4), 0.6, 0.1373, [0.0009, -0.0009], 1.5, 2, 4, False),  # 4 blocks per axis
    ((16, 8, 16, 24), (4, 4, 4, 4), 0.6, 0.1373, [0.0009], 1.5, 2, 4, True),   # 4, 2, 4, 6 blocks per axis
]


@pytest.fixture(scope="module")
def fields():
    out = []
    for k, (dims, bd, eps, kappa, mus, csw, cyc, mr, ap) in enumerate(CASES):
        U = synth.gauge_field(dims, eps, seed=30 + k)
        b = synth.gaussian_spinor(dims, len(mus), seed=130 + k)
        x0 = 0.1 * synth.gaussian_spinor(dims, len(mus), seed=230 + k)
        op = oracle.Operator(dims, U, oracle.kappa_to_m(kappa), 0.0, csw, antiperiodic_t=ap)
        ref = np.stack([op.with_mu(m).sap(b[i], bd, cyc, mr, x0=x0[i]).reshape(-1, 4, 3)
                        for i, m in enumerate(mus)])
        out.append((U, b, x0, ref))
    return out


@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_sap_matches_oracle(fields, case, prec):
    dims, bd, eps, kappa, mus, csw, cyc, mr, ap = CASES[case]
    U, b, x0, ref = fields[case]
    announce(f"sap parity case={case} dims={dims} block={bd} prec={prec}")
    x = dev(x0)
    tm.tm_sap_smooth(dims, dev(U), dev(b), x, kappa, mus, csw, bd, cyc, mr, storage=prec, antiperiodic_t=ap)
    got = host(x)
    for i in range(len(mus)):
        check_close(got[i], ref[i], "sap", prec, f"case {case} {dims} block {bd} system {i}")


def test_sap_many_systems_match_single(fields):
    # 12 systems (+-mu) in one launch give the same result as one system at a time
    dims, bd, eps, kappa, mus, csw, cyc, mr, ap = CASES[1]
    U, _, _, _ = fields[1]
    announce("sap 12 systems vs single")
    b = synth.gaussian_spinor(dims, 12, seed=77)
    mus12 = [0.003 if k % 2 == 0 else -0.003 for k in range(12)]
    x = dev(np.zeros_like(b))
    tm.tm_sap_smooth(dims, dev(U), dev(b), x, kappa, mus12, csw, bd, 2, 4, storage="f32")
    allx = host(x)
    for k in (0, 5, 11):
        xs = dev(np.zeros_like(b[k:k + 1]))
        tm.tm_sap_smooth(dims, dev(U), dev(b[k:k + 1]), xs, kappa, [mus12[k]], csw, bd, 2, 4, storage="f32")
        assert np.array_equal(host(xs)[0], allx[k])


def test_sap_error_paths(fields):
    dims, bd, eps, kappa, mus, csw, cyc, mr, ap = CASES[1]
    U, b, x0, _ = fields[1]
    announce("sap error paths")
    x = dev(x0)
    with pytest.raises(tm.TMError) as e:
        tm.tm_sap_smooth(dims, dev(U), dev(b), x, kappa, mus, csw, (8, 4, 4, 4), cyc, mr)
    assert e.value.code == -3  # one block along t
    with pytest.raises(tm.TMError) as e:
        tm.tm_sap_smooth(dims, dev(U), dev(b), x, kappa, mus, csw, (3, 4, 4, 4), cyc, mr)
    assert e.value.code == -2
    z16 = dev(np.zeros((len(mus), 16 ** 4, 4, 3)))
    with pytest.raises(tm.TMError) as e:
        tm.tm_sap_smooth((16, 16, 16, 16), dev(np.zeros((16 ** 4, 4, 3, 3))), z16, z16.clone(), kappa, mus, csw,
                         (8, 8, 8, 4), cyc, mr)
    assert e.value.code == -3  # 2048-site block
    # buffers that do not match the lattice and the systems are refused before the library is called
    with pytest.raises(ValueError):
        tm.tm_sap_smooth(dims, dev(U), dev(b[:1]), x, kappa, mus, csw, bd, cyc, mr)


@pytest.mark.parametrize("prec,bd,tiny", [("f32", (4, 4, 4, 4), 1e-21), ("f32", (4, 4, 2, 4), 1e-21),
                                          ("f16", (4, 4, 4, 4), 1e-21), ("bf16", (4, 4, 4, 4), 1e-21),
                                          ("f32", (4, 4, 4, 8), 1e-21), ("f16", (4, 4, 4, 4), 1e-40),
                                          ("f32", (4, 4, 4, 4), 1e-40)])
def test_sap_blocks_with_vanishing_residual(prec, bd, tiny):
    # Far from a point source the block residuals shrink below the smallest
    # normal FP32 number once squared; such blocks must keep e (a step length
    # from a subnormal <q,q> is inf or NaN).  One O(1) site, every other
    # component ~1e-21, so <q,q> ~ 1e-39 in the other blocks; at 1e-40 the
    # fields themselves are FP32 subnormals (the FP16 per-site scale too).
    dims, kappa, mu, csw = (8, 8, 8, 16), 0.1373, 0.0009, 1.5
    U = synth.gauge_field(dims, 0.6, seed=21)
    b = tiny * synth.gaussian_spinor(dims, 1, seed=121)
    b[0, 0, 0, 0] = 1.0
    announce(f"sap vanishing residual prec={prec} block={bd} tiny={tiny}")
    x = dev(np.zeros_like(b))
    tm.tm_sap_smooth(dims, dev(U), dev(b), x, kappa, [mu], csw, bd, 2, 4, storage=prec)
    got = host(x)[0]
    assert np.isfinite(got).all()
    op = oracle.Operator(dims, U, oracle.kappa_to_m(kappa), mu, csw)
    ref = op.sap(b[0], bd, 2, 4).reshape(-1, 4, 3)
    check_close(got, ref, "sap", prec, f"vanishing residual block {bd} tiny {tiny}")


@pytest.mark.parametrize("prec", ["f32", "f16"])
def test_sap_without_mr_steps_leaves_x(prec):
    # zero MR steps: every block's correction is zero, so x comes back as stored (rounded once to
    # the storage precision) whatever the number of cycles; several systems run through the 4^4
    # kernel's system loop with no MR step between one system's residual and the next one's
    dims, bd = (8, 8, 8, 8), (4, 4, 4, 4)
    U = synth.gauge_field(dims, 0.5, seed=41)
    mus = [0.003, -0.003, 0.01]
    b = synth.gaussian_spinor(dims, len(mus), seed=141)
    x0 = synth.gaussian_spinor(dims, len(mus), seed=241)
    announce(f"sap with mr_iters 0, {prec}")
    Ud = dev(U)
    outs = []
    for cyc in (1, 3):
        x = dev(x0)
        tm.tm_sap_smooth(dims, Ud, dev(b), x, 0.16, mus, 1.5, bd, cyc, 0, storage=prec)
        outs.append(host(x))
    assert np.array_equal(outs[0], outs[1])
    bound = 1e-6 if prec == "f32" else 1e-3
    for i in range(len(mus)):
        assert rel_err(outs[0][i], x0[i]) < bound, i


# Squares below the smallest normal number in the FP64 and the even-odd kernels, on 4^4 blocks (two lanes per site) and
# others: 1e-160 squared for FP64, 1e-21 for FP32 (1e-40: fields that are FP32 subnormals themselves).
@pytest.mark.parametrize("prec,eo,bd,tiny", [("f64", False, (4, 4, 4, 4), 1e-160), ("f64", True, (4, 4, 4, 4), 1e-160),
                                             ("f32", True, (4, 4, 4, 4), 1e-21), ("f32", True, (4, 4, 4, 4), 1e-40),
                                             ("bf16", True, (4, 4, 4, 4), 1e-21), ("f64", False, (4, 4, 4, 2), 1e-160),
                                             ("f64", False, (4, 4, 4, 8), 1e-160), ("f64", True, (2, 2, 2, 2), 1e-160),
                                             ("f32", True, (4, 4, 4, 8), 1e-21)])
def test_sap_kernels_with_vanishing_residual(prec, eo, bd, tiny):
    dims, kappa, mu, csw = (8, 8, 8, 16), 0.1373, 0.0009, 1.5
    U = synth.gauge_field(dims, 0.6, seed=22)
    b = tiny * synth.gaussian_spinor(dims, 1, seed=122)
    b[0, 0, 0, 0] = 1.0
    announce(f"sap vanishing residual prec={prec} eo={eo} block={bd} tiny={tiny}")
    x = dev(np.zeros_like(b))
    tm.tm_sap_smooth(dims, dev(U), dev(b), x, kappa, [mu], csw, bd, 2, 4, storage=prec, eo=eo)
    got = host(x)[0]
    assert np.isfinite(got).all()
    ref = oracle.Operator(dims, U, oracle.kappa_to_m(kappa), mu, csw).sap(b[0], bd, 2, 4, eo=eo).reshape(-1, 4, 3)
    check_close(got, ref, "sap", prec, f"vanishing residual eo {eo} block {bd} tiny {tiny}")


# All systems of a call in one workgroup, with no MR step or a few between one system's residual and the next one's:
# each kernel's own system loop, against one system per call.
@pytest.mark.parametrize("mr", [0, 3])
@pytest.mark.parametrize("bd", [(2, 2, 2, 2), (4, 4, 4, 2), (4, 4, 4, 4), (4, 4, 4, 8)])
@pytest.mark.parametrize("prec,eo", [("f64", False), ("f32", False), ("bf16", False), ("f64", True), ("f32", True)])
def test_systems_in_one_workgroup_match_single_calls(prec, eo, bd, mr):
    dims, mus = (8, 8, 8, 16), [0.003, -0.003, 0.02, -0.02]
    U, b = dev(synth.gauge_field(dims, 0.5, seed=42)), synth.gaussian_spinor(dims, len(mus), seed=142)
    announce(f"systems in one workgroup prec={prec} eo={eo} block={bd} mr={mr}")

    def smooth(k0, k1):
        x = dev(0.1 * b[k0:k1])
        tm.tm_sap_smooth(dims, U, dev(b[k0:k1]), x, 0.1373, mus[k0:k1], 1.5, bd, 2, mr, storage=prec, eo=eo,
                         sys_tile=k1 - k0, gauge_tag=3)
        return host(x)

    together = smooth(0, len(mus))
    for k in range(len(mus)):
        assert np.array_equal(together[k], smooth(k, k + 1)[0]), k
    if mr == 0 and not eo:  # no correction: x as stored
        assert rel_err(together, 0.1 * b) < {"f64": 1e-15, "f32": 1e-7, "bf16": 4e-3}[prec]
