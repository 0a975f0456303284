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
