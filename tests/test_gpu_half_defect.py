"""The defect of a float32 pre-smoothing pass, one value per pair of vertices,
and its restriction, against the oracle: partial coarse tiles (4 x 64), chunks
that end inside a group of eight planes, padded rows (finest level) and dense
odd ones (below it), both colour orders and face means."""
import numpy as np
import pytest

from gpu_util import dev, host, rel_max, say
from test_gpu_kernels import defect_scale, make, oracle_pre

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,face_mean", [(96, "arith"), (96, "harmonic"), (128, "harmonic"), (192, "arith")])
@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("wgs", ["16", "512"])
def test_half_defect_restriction(N, face_mean, order, wgs, monkeypatch):
    import torch
    from paper_2608_00760_amd import synth
    say("half defect N=%d %s order=%d wgs=%s" % (N, face_mean, order, wgs))
    monkeypatch.setenv("DMGS_SWEEP2_MIN", "32")
    monkeypatch.setenv("DMGS_DR_WGS", wgs)
    P, H = make(N, 40 + N, precision="fp32-in-fp64", face_mean=face_mean)
    for k in range(P.levels - 1):
        if H.Ns[k] < 32:
            break
        f32 = lambda a: a.astype(np.float32).astype(np.float64)
        u, q = f32(synth.normal(H.Ns[k], 1 + k)), f32(synth.normal(H.Ns[k], 2 + k))
        gu, gqc = P.debug_pre(k, dev(u, torch.float32), dev(q, torch.float32), order=order, fp32=True)
        ru, rqc = oracle_pre(H, k, u, q, order)
        # the tolerances of the float32 passes' own tests
        assert rel_max(host(gu), ru) <= 2e-5, (k, "pre u")
        assert np.abs(host(gqc) - rqc).max() <= 2e-5 * defect_scale(H, k, ru, q), (k, "pre qc")


@pytest.mark.parametrize("precision,face_mean", [("fp32-in-fp64", "arith"), ("fp32-in-fp64", "harmonic"),
                                                 ("fp64", "arith"), ("fp64", "harmonic")])
@pytest.mark.parametrize("order", [0, 1])
def test_results_do_not_depend_on_chunks(precision, face_mean, order, monkeypatch):
    """Two-sweep passes cut into one, a few and many chunks: the same bits
    (grouped execution chooses the chunks for the group)."""
    import torch
    from paper_2608_00760_amd import synth
    N, fp32 = 96, precision != "fp64"
    say("chunks %s %s order=%d" % (precision, face_mean, order))
    monkeypatch.setenv("DMGS_SWEEP2_MIN", "32")
    t = torch.float32 if fp32 else torch.float64
    ref = None
    for wgs in ("16", "40", "256"):
        monkeypatch.setenv("DMGS_SWEEP2_WGS", wgs)
        P, H = make(N, 7, precision=precision, face_mean=face_mean)
        u, q, ec = (dev(synth.normal(n, i), t) for i, n in ((1, N), (2, N), (3, N // 2)))
        got = [*P.debug_pre(0, u, q, order=order, fp32=fp32), P.debug_post(0, u, ec, q, order=order, fp32=fp32)]
        if ref is None:
            ref = got
        for a, b in zip(got, ref):
            assert torch.equal(a, b), wgs
