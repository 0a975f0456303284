"""General grids of more tiles than the other reductions have parts.

The residual norm rides on the block passes up to 4096 tiles of 8^3: on grids
of 1280, 3456 and 4096 tiles each tolerance solve launches its residual pass
once (the initial norm), above (5120) once a cycle too, and the reported norm
is the oracle operator's of the returned iterate (1e-3 of it, as in the other
tests of that norm: one of the wrong iterate or colour, or without a share of
its parts, is off by more).  The likelihood's sums, with the epilogue on the
block passes or after them, equal numpy's from the returned rho (1e-12: both
are float64 sums of positive terms).
"""
import numpy as np
import pytest

from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [(32, 64, 32), (160, 64, 64), (192, 96, 96), (256, 128, 64), (320, 128, 64)])
def test_norm_and_epilogue_on_many_tiles(cells):
    from oracle import likelihood, refgrid
    from paper_2608_00760_amd import synth
    from paper_2608_00760_amd.solver import Options, Plan
    tiles = int(np.prod([(n + 7) // 8 for n in cells]))
    say("many tiles", cells, tiles)
    c = synth.grid_case(cells, 1500)
    h = tuple(float(a) for a in (7.5 / cells[0], 3.5 / cells[1], 3.5 / cells[2]))
    P = Plan(Options(cells[0], shape=cells, spacing=h))
    P.set_log_coefficients(dev(c["logD"]), dev(c["logmua"]))
    P.timing(True)
    rho, info = P.forward(dev(c["q"]))
    (qbar, _, _), vi = P.vjp(rho, dev(c["rhobar"]), coef_grads=False)
    n = P.timing_read()["residual"]["launches"]
    P.timing(False)
    say("  cycles %d + %d, residual passes %d" % (info["cycles"], vi["cycles"], n))
    H = refgrid.HierarchyGrid(c["D"], c["mua"], h=h)
    for x, b, i in ((rho, c["q"], info), (qbar, c["rhobar"], vi)):
        rel = np.linalg.norm(H.defect(0, host(x), b)) / np.linalg.norm(H.defect(0, np.zeros_like(b), b))
        assert i["rel_residual"] <= 1e-10 and abs(rel - i["rel_residual"]) <= 1e-3 * i["rel_residual"]
    assert n == (2 if tiles <= 4096 else 2 + info["cycles"] + vi["cycles"])
    Le = c["mua"] * host(rho)
    w = likelihood.noise_weights(np.abs(Le), 3)
    d = Le + 0.05 * np.abs(Le) * np.random.default_rng(1501).standard_normal(Le.shape)
    (rho2, val, _), fi, _ = P.likelihood_grad(dev(c["q"]), dev(d), dev(w))
    assert np.array_equal(host(rho2), host(rho)) and fi["cycles"] == info["cycles"]
    rH, rchi2, rn = likelihood.neg_log_likelihood(host(rho2), c["mua"], d, w)
    assert val["nvox"] == rn and abs(val["H"] - rH) <= 1e-12 * rH and abs(val["chi2"] - rchi2) <= 1e-12 * rchi2
    P.close()
