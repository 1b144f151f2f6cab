"""The schedules of quantize_layer: which one a layer takes, and that they agree."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import DEV, note, rel_frob, rot_device, to_np
from paper_2607_07964_amd import layer as L


def test_schedule_rule():
    """Two streams (a long H_G after the transforms) until H_G outlasts the rest 15 times."""
    for tokens, d_out, d_in, late, one in (
            (262144, 4096, 4096, False, False), (262144, 4096, 14336, False, False),
            (65536, 14336, 4096, False, False), (262144, 14336, 4096, True, False),
            (131072, 28672, 8192, True, False), (262144, 28672, 8192, True, True),
            (131072, 28672, 4096, True, True), (2048, 256, 256, False, False)):
        assert L._cov_late(tokens, d_out, d_in) == late
        assert L._one_stream(tokens, d_out, d_in) == one


@pytest.mark.gpu
@pytest.mark.parametrize("late,one,cus", [(False, False, None), (True, False, None),
                                          (True, True, None), (True, True, 64)])
def test_schedules_agree(monkeypatch, late, one, cus):
    """Each schedule against the serial calls: the same but for the order of H_G's sums."""
    spec = synth.small_spec(448, 256, 4096, bits=4, seed=11)
    X, G, W0 = (synth.gen_matrix(m, DEV) for m in (spec.x, spec.g, spec.w))
    rin, rout = (rot_device(synth.rotation_params(d, 3, s))
                 for d, s in ((spec.d_in, "in"), (spec.d_out, "out")))
    outs = []
    for overlap in (False, True):
        if overlap:
            monkeypatch.setattr(L, "_cov_late", lambda *a: late)
            monkeypatch.setattr(L, "_one_stream", lambda *a: one)
        st = L.LayerState.allocate(spec.d_out, spec.d_in, spec.n_tokens, DEV, x_dtype=X.dtype,
                                   g_dtype=G.dtype)
        note(f"schedule late={late} one={one} cus={cus} {L.schedule(st, spec.n_tokens, overlap, cus)}")
        assert (L.schedule(st, spec.n_tokens, overlap, cus) == "one stream") == (
            not overlap or (one and cus is None))
        for _ in range(2):  # (the second time over the first's results)
            L.quantize_layer(st, X, G, W0, rin, rout, spec.bits, overlap=overlap, cov_cus=cus)
        torch.cuda.synchronize()
        outs.append(st)
    a, b = outs
    for f in ("codes", "W", "U", "HX", "sx", "sg", "scales", "zeros"):
        assert np.array_equal(to_np(getattr(a, f)), to_np(getattr(b, f))), f
    # two orders of 4096-token fp32 sums, each within 4096 2^-24 of the terms
    assert rel_frob(to_np(b.HG), to_np(a.HG)) < 1e-5
    np.testing.assert_allclose(to_np(b.tr_pre), to_np(a.tr_pre), rtol=1e-5)
    np.testing.assert_allclose(to_np(b.tr_post), to_np(a.tr_post), rtol=1e-5)
