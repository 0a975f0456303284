"""Norms added up by the launch's last workgroup, with many parts.

Float64 tolerance solves whose norm has 216 and 256 parts from block passes
and 216 to 504 from marching ones, each repeated beside another plan's solves
on a stream and thread of their own: every solve leaves the same bits in its
whole residual history (a part missed, taken twice or read before it was
stored would change them), and the last entry is the oracle operator's
residual of the result (1e-3 of it, as in the other tests of these norms).
"""
import threading

import numpy as np
import pytest

from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [48, (64, 32, 64), 96, 128, 192])
def test_norm_of_many_parts_repeats(cells, monkeypatch):
    import torch
    from oracle import ref, refgrid
    from paper_2608_00760_amd import synth
    from paper_2608_00760_amd.solver import Options, Plan
    say("norm parts", cells)
    monkeypatch.setenv("DMGS_TRACE", "1")
    if isinstance(cells, tuple):
        c = synth.grid_case(cells, 1700)
        H = refgrid.HierarchyGrid(c["D"], c["mua"])
        P = Plan(Options(cells[0], shape=cells))
    else:
        c = synth.grf_case(cells, 1700 + cells)
        H = ref.Hierarchy(c["D"], c["mua"])
        P = Plan(Options(cells))
    P.set_coefficients(dev(c["D"]), dev(c["mua"]))
    other = synth.grf_case(32, 1799)
    Q = Plan(Options(32))
    Q.set_coefficients(dev(other["D"]), dev(other["mua"]))
    q, oq = dev(c["q"]), dev(other["q"])
    torch.cuda.synchronize()
    stop, count = threading.Event(), [0]

    def beside():
        with torch.cuda.stream(torch.cuda.Stream()):
            while not stop.is_set():
                Q.forward(oq)
                count[0] += 1

    th = threading.Thread(target=beside)
    th.start()
    try:
        first = None
        for _ in range(20):
            rho, info = P.forward(q)
            tr = P.trace(0)
            first = first or tr
            assert tr == first
    finally:
        stop.set()
        th.join()
    assert count[0] > 0
    b = c["q"]
    rel = np.linalg.norm(H.defect(0, host(rho), b)) / np.linalg.norm(H.defect(0, np.zeros_like(b), b))
    say("  cycles %d, rel %.3e (oracle %.3e), %d solves beside" % (info["cycles"], info["rel_residual"], rel, count[0]))
    assert abs(rel - info["rel_residual"]) <= 1e-3 * info["rel_residual"]
    P.close()
    Q.close()
