"""The no-allocation smoother tm_sap_smooth_noalloc against tm_sap_smooth.

Both entry points run the same kernels on the same inputs, so the results must
agree bit for bit.  Two calls in a row, the second on a smaller lattice with
fewer systems, check that the fixed scratch array's leftovers from the first
call do not leak into the second.  A problem larger than the array is refused
before any device work.
"""
import numpy as np
import pytest

import oracle
import paper_1610_02370_amd as tm
from paper_1610_02370_amd import synth

from gpu_util import announce, check_close, dev, host

pytestmark = pytest.mark.gpu

CALLS = [
    # dims, block, storage, mus, cycles, mr, io
    ((8, 8, 8, 8), (4, 4, 4, 4), "f32", [0.003, -0.003], 2, 4, "canonical"),
    ((4, 4, 4, 8), (2, 2, 2, 2), "f32", [0.01], 2, 3, "canonical"),
    ((8, 8, 4, 8), (4, 4, 2, 4), "f64", [0.001, -0.002], 1, 4, "canonical"),
    ((4, 4, 4, 4), (2, 2, 2, 2), "f16", [0.01], 2, 4, "internal"),
]


def run_both(dims, block, storage, mus, cyc, mr, io, seed):
    import torch

    kappa, csw = 0.1373, 1.5
    U = synth.gauge_field(dims, 0.5, seed=seed)
    b = synth.gaussian_spinor(dims, len(mus), seed=100 + seed)
    x0 = 0.1 * synth.gaussian_spinor(dims, len(mus), seed=200 + seed)
    out = []
    for fn in (tm.tm_sap_smooth, tm.tm_sap_smooth_noalloc):
        if io == "canonical":
            x = dev(x0)
            fn(dims, dev(U), dev(b), x, kappa, mus, csw, block, cyc, mr, storage=storage)
            out.append(host(x))
        else:
            n = tm.tm_spinor_bytes(dims, len(mus), storage, layout_block=block)
            bi = torch.zeros(n, dtype=torch.uint8, device="cuda")
            xi = torch.zeros(n, dtype=torch.uint8, device="cuda")
            tm.tm_spinor_import(dims, dev(b), bi, storage=storage, layout_block=block)
            tm.tm_spinor_import(dims, dev(x0), xi, storage=storage, layout_block=block)
            fn(dims, dev(U), bi, xi, kappa, mus, csw, block, cyc, mr, storage=storage, io="internal")
            x = dev(np.zeros_like(x0))
            tm.tm_spinor_export(dims, xi, x, storage=storage, layout_block=block)
            out.append(host(x))
    torch.cuda.synchronize()
    op = oracle.Operator(dims, U, oracle.kappa_to_m(kappa), 0.0, csw)
    refs = [op.with_mu(m).sap(b[i], block, cyc, mr, x0=x0[i]).reshape(-1, 4, 3) for i, m in enumerate(mus)]
    return out[0], out[1], refs


def test_noalloc_matches_sap_smooth_on_successive_calls():
    for k, (dims, block, storage, mus, cyc, mr, io) in enumerate(CALLS):
        announce(f"no-alloc call {k}: dims={dims} block={block} storage={storage} systems={len(mus)} io={io}")
        ref_entry, got, refs = run_both(dims, block, storage, mus, cyc, mr, io, seed=50 + k)
        assert np.isfinite(got).all()
        assert np.array_equal(got, ref_entry), k
        for i in range(len(mus)):
            check_close(got[i], refs[i], "sap", storage, f"no-alloc call {k} system {i}")


def test_noalloc_refuses_problems_beyond_its_scratch():
    import torch

    dims = (16, 16, 16, 16)
    V = 16 ** 4
    announce("no-alloc size limit")
    U = torch.zeros((V, 4, 3, 3), dtype=torch.complex128, device="cuda")
    b = torch.zeros((4, V, 4, 3), dtype=torch.complex128, device="cuda")
    x = torch.zeros_like(b)
    # 16^4 sites at FP32 with 4 systems: 65536 * (480 + 4 * 192) bytes > 64 MiB
    with pytest.raises(tm.TMError) as e:
        tm.tm_sap_smooth_noalloc(dims, U, b, x, 0.15, [0.1] * 4, 1.0, (4, 4, 4, 4), 1, 1, storage="f32")
    assert e.value.code == -1 and "scratch" in str(e.value)
    with pytest.raises(tm.TMError) as e:
        tm.tm_sap_smooth_noalloc(dims, U, b[:1], x[:1], 0.15, [0.1], 1.0, (4, 4, 4, 4), 1, 1, storage="f64")
    assert e.value.code == -1


# The clover term built from the canonical links, with no staged copy (tm_sap_smooth stages them): boxes of the build
# cut off by the lattice's end, extents in steps of 3 and of 4.
@pytest.mark.parametrize("dims,block", [((6, 10, 6, 14), (3, 5, 3, 7)), ((2, 6, 10, 6), (1, 3, 5, 3)), ((10, 2, 6, 14), (5, 1, 3, 7))])
def test_noalloc_builds_the_clover_term_without_staging(dims, block):
    announce(f"no-alloc clover build dims={dims} block={block}")
    a, b, ref = run_both(dims, block, "f64", [0.002], 1, 2, "canonical", 61)
    assert np.array_equal(a, b)
    check_close(b[0], ref[0], "sap", "f64", f"no-alloc clover build {dims}")
