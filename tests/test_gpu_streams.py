"""Calls on two streams of one device: what a call on internal buffers may overlap (tm.h, streams)."""
import pytest

import paper_1610_02370_amd as tm
from paper_1610_02370_amd import synth

from gpu_util import announce, dev

pytestmark = pytest.mark.gpu


def test_gauge_build_leaves_a_canonical_call_on_another_stream_alone():
    # a smoother on canonical buffers is still at work on one stream while a call on internal buffers takes in other
    # links on a second one: the build's staged links must not land in the first call's workspace
    import torch

    dims, nsys = (16, 16, 16, 16), 12
    mus = [0.01 * (k + 1) for k in range(nsys)]
    U, V = (dev(synth.gauge_field(dims, 0.5, seed=s)) for s in (31, 32))
    b = dev(synth.gaussian_spinor(dims, nsys, seed=131))
    announce("gauge build beside a canonical smoother")

    def smooth(x, stream=None):
        tm.tm_sap_smooth(dims, U, b, x, 0.1373, mus, 1.5, (4, 4, 4, 4), 30, 4, storage="f32", gauge_tag=5, stream=stream)

    n = tm.tm_spinor_bytes(dims, 1, "f64")
    p, q, alone = (torch.zeros(n // 8, dtype=torch.float64, device="cuda") for _ in range(3))
    tm.tm_spinor_import(dims, b[:1].contiguous(), p, storage="f64")
    ref, x = torch.zeros_like(b), torch.zeros_like(b)
    smooth(ref)
    tm.tm_dirac_apply(dims, V, p, 0.1373, [0.01], 1.5, out=alone, io="internal")
    torch.cuda.synchronize()
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    smooth(x, one)
    tm.tm_dirac_apply(dims, V, p, 0.1373, [0.01], 1.5, out=q, io="internal", stream=two)
    torch.cuda.synchronize()
    assert torch.equal(x, ref)
    assert torch.equal(q, alone)
