"""General grids of more tiles than the other reductions have parts.

The likelihood's epilogue and the residual norm ride on the block passes
whatever the number of 8^3 tiles: on grids of 1280 and 3456 tiles (the data
grid has 1024) the fused solve equals the one with the separate epilogue pass
as on small grids, each tolerance solve launches its residual pass once (the
initial norm), and the reported norm is the oracle operator's of the returned
iterate (1e-3 of it, as in the other tests of that norm: one of the wrong
iterate or colour, or without a share of its parts, is off by more).
"""
import numpy as np
import pytest

from gpu_util import dev, host, say
from test_gpu_likelihood import fused_vs_separate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [(160, 64, 64), (192, 96, 96)])
def test_epilogue_and_norm_on_many_tiles(cells, monkeypatch):
    import torch
    from oracle import refgrid
    from paper_2608_00760_amd import synth
    from paper_2608_00760_amd.solver import Options, Plan
    say("many tiles", cells)
    c = synth.grid_case(cells, 1500)
    h = tuple(float(a) for a in (7.5 / cells[0], 3.5 / cells[1], 3.5 / cells[2]))

    def make():
        P = Plan(Options(cells[0], shape=cells, spacing=h))
        P.set_log_coefficients(dev(c["logD"]), dev(c["logmua"]))
        return P
    P = make()
    P.timing(True)
    rho, info = P.forward(dev(c["q"]))
    (qbar, _, _), vi = P.vjp(rho, dev(c["rhobar"]), coef_grads=False)
    n = P.timing_read()["residual"]["launches"]
    say("  cycles %d + %d, residual passes %d" % (info["cycles"], vi["cycles"], n))
    H = refgrid.HierarchyGrid(c["D"], c["mua"], h=h)
    for x, b, i in ((rho, c["q"], info), (qbar, c["rhobar"], vi)):
        rel = np.linalg.norm(H.defect(0, host(x), b)) / np.linalg.norm(H.defect(0, np.zeros_like(b), b))
        assert i["rel_residual"] <= 1e-10 and abs(rel - i["rel_residual"]) <= 1e-3 * i["rel_residual"]
    assert n == 2
    Le = c["mua"] * host(rho)
    w = host(P.noise_weights(dev(np.abs(Le)), 3))
    P.close()
    sigma = np.sqrt(np.where(w > 0, 1.0 / np.where(w > 0, w, 1.0), 0.0))
    d = Le + sigma * np.random.default_rng(1501).standard_normal(Le.shape)
    fused_vs_separate(make, c["q"], d, w, 0, monkeypatch)
