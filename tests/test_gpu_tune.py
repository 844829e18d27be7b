"""GPU tests of the SAP tuner and of splitting systems over workgroups.

Systems are independent in every SAP step, so the split of a batch over
workgroups must not change a single bit of the result.  The tuner's choice is
checked for validity and round-tripped through its cache; a solve that asks
for the cached shape (block_dims all zero) must still reach the requested
true residual, and SAP with the tuned shape is compared with the oracle run
on the same shape.
"""
import numpy as np
import pytest

import oracle
import paper_1610_02370_amd as tm
from paper_1610_02370_amd import synth

from gpu_util import announce, dev, host, rel_err

pytestmark = pytest.mark.gpu

DIMS = (8, 8, 8, 16)
KAPPA, CSW = 0.1373, 1.5


@pytest.fixture(scope="module")
def field():
    return synth.gauge_field(DIMS, 0.6, seed=61)


@pytest.mark.parametrize("prec", ["f32", "f16", "f64"])
def test_sys_tile_is_bit_identical(field, prec):
    mus = [0.0009 * (1 if k % 2 == 0 else -1) for k in range(6)]
    b = synth.gaussian_spinor(DIMS, 6, seed=161)
    announce(f"sys_tile split prec={prec}")
    out = []
    for tile in (0, 1, 4):
        x = dev(np.zeros_like(b))
        tm.tm_sap_smooth(DIMS, dev(field), dev(b), x, KAPPA, mus, CSW, (4, 4, 4, 4), 2, 4, storage=prec,
                         sys_tile=tile)
        out.append(host(x))
    assert np.array_equal(out[0], out[1])
    assert np.array_equal(out[0], out[2])


@pytest.mark.parametrize("prec,dims,nsys", [("f32", (8, 8, 8, 8), 12), ("f64", (8, 8, 8, 8), 5), ("f64", (3, 5, 2, 7), 4),
                                            ("f32", (6, 4, 2, 5), 3)])
def test_split_application_is_bit_identical(prec, dims, nsys):
    # lattices with far fewer tiles than the device holds: the systems of one call go to several
    # workgroups per tile and give what one system at a time gives
    mus = [0.01 * (k + 1) for k in range(nsys)]
    U, psi = synth.gauge_field(dims, 0.6, seed=62), synth.gaussian_spinor(dims, nsys, seed=162)
    announce(f"application split prec={prec} dims={dims}")
    got = host(tm.tm_dirac_apply(dims, dev(U), dev(psi), KAPPA, mus, CSW, storage=prec))
    for k in range(nsys):
        one = host(tm.tm_dirac_apply(dims, dev(U), dev(psi[k:k + 1]), KAPPA, [mus[k]], CSW, storage=prec))
        assert np.array_equal(got[k], one[0])


def test_autotune_round_trip(field, tmp_path, monkeypatch):
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("TM_TUNE_CACHE", str(cache))
    mus = [0.0009, -0.0009]
    announce("autotune f32 dims=%s nsys=2" % (DIMS,))
    block, tile = tm.tm_autotune_sap(DIMS, dev(field), KAPPA, mus, CSW, 2, 4, storage="f32")
    vb = int(np.prod(block))
    assert 16 <= vb <= 256
    for d, l in zip(DIMS, block):
        assert d % l == 0 and (d // l) % 2 == 0
    assert tile in (0, 1)
    lines = cache.read_text().splitlines()
    assert len(lines) == 1
    key, choice = lines[0].split(" : ")
    assert key.split()[:6] == ["sap", *map(str, DIMS), "2"]
    assert tuple(map(int, choice.split()[:4])) == tuple(block)

    # SAP with the tuned shape against the oracle on the same shape
    b = synth.gaussian_spinor(DIMS, 2, seed=162)
    x = dev(np.zeros_like(b))
    tm.tm_sap_smooth(DIMS, dev(field), dev(b), x, KAPPA, mus, CSW, block, 2, 4, storage="f32", sys_tile=tile)
    op = oracle.Operator(DIMS, field, oracle.kappa_to_m(KAPPA), 0.0, CSW)
    got = host(x)
    for i, m in enumerate(mus):
        ref = op.with_mu(m).sap(b[i], block, 2, 4).reshape(-1, 4, 3)
        assert rel_err(got[i], ref) < 2e-4

    # a solve that takes the cached shape
    xs = dev(np.zeros_like(b))
    rc, rep = tm.tm_fgmres_solve(DIMS, dev(field), dev(b), xs, KAPPA, mus, CSW, 1e-10, storage="f32",
                                 block_dims=(0, 0, 0, 0), n_cycles=2, mr_iters=4)
    assert rc == 0
    assert max(rep["true_rel_res"][:2]) <= 1e-10
    for i, m in enumerate(mus):
        r = op.with_mu(m).apply(host(xs)[i]) - b[i].reshape(-1, 4, 3)
        assert np.linalg.norm(r) / np.linalg.norm(b[i]) <= 1.5e-10


def test_autotune_rejects_bad_input(field, tmp_path, monkeypatch):
    monkeypatch.setenv("TM_TUNE_CACHE", str(tmp_path / "t.txt"))
    announce("autotune error paths")
    with pytest.raises(tm.TMError):
        tm.tm_autotune_sap(DIMS, dev(field), KAPPA, [0.0], CSW, 0, 4, storage="f32")
    with pytest.raises(tm.TMError):
        # no block of 16..256 sites with an even block count fits a 2^4 lattice
        tm.tm_autotune_sap((2, 2, 2, 2), dev(synth.gauge_field((2, 2, 2, 2), 0.3, seed=1)), KAPPA, [0.0], CSW, 1, 4,
                           storage="f32")
    assert not (tmp_path / "t.txt").exists()
