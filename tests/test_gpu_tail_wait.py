"""The coarse kernel's bounded wait for the other workgroups of its launch.

With the bound at 0 (DMGS_TAIL_SPINS) the wait gives up at once, in every
form: both precisions, one coarse level (the matrix alone) and several, cubic
and general grids, the pull-back and grouped execution.  Every workgroup ends
and the solve reports a non-finite residual, on this call and the next, and
other plans solve as ever.
"""
import numpy as np
import pytest

from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


def make(cells, precision, face_mean="arith"):
    from paper_2608_00760_amd import synth
    from paper_2608_00760_amd.solver import Options, Plan
    if isinstance(cells, tuple):
        c = synth.grid_case(cells, 1600)
        P = Plan(Options(cells[0], shape=cells, face_mean=face_mean))
    else:
        c = synth.grf_case(cells, 1600 + cells)
        P = Plan(Options(cells, precision=precision, face_mean=face_mean))
    P.set_coefficients(dev(c["D"]), dev(c["mua"]))
    return P, c


@pytest.mark.parametrize("cells,precision", [(8, "fp64"), (32, "fp64"), (48, "fp64"), (32, "fp32-in-fp64"),
                                             (64, "fp32-in-fp64"), ((16, 8, 8), "fp64"), ((64, 32, 32), "fp64")])
@pytest.mark.parametrize("face_mean", ["arith", "harmonic"])
def test_wait_given_up(cells, precision, face_mean, monkeypatch):
    from paper_2608_00760_amd import _abi
    say("tail wait", cells, precision, face_mean)
    good, c = make(cells, precision, face_mean)
    ref, _ = good.forward(dev(c["q"]))
    monkeypatch.setenv("DMGS_TAIL_SPINS", "0")
    bad, _ = make(cells, precision, face_mean)
    monkeypatch.delenv("DMGS_TAIL_SPINS")
    for _ in range(2):
        with pytest.raises(_abi.DMGSError) as e:
            bad.forward(dev(c["q"]))
        assert e.value.status == _abi.DMGS_ERR_NONFINITE
        with pytest.raises(_abi.DMGSError) as e:
            bad.vjp(ref, dev(c["rhobar"]))
        assert e.value.status == _abi.DMGS_ERR_NONFINITE
        again, _ = good.forward(dev(c["q"]))
        assert np.array_equal(host(again), host(ref))
    bad.close()
    good.close()


def test_wait_given_up_in_a_group(monkeypatch):
    """One request of three gives up: it fails, the others' bits are their own."""
    import test_gpu_batch as batch
    from paper_2608_00760_amd import _abi
    from paper_2608_00760_amd.solver import Batch
    say("tail wait, grouped")
    B, reqs = Batch(), {}
    for tag, N in enumerate((64, 64, 96)):
        if tag == 1:
            monkeypatch.setenv("DMGS_TAIL_SPINS", "0")
        P, c, t = batch.make_plan(N, 30 + tag)
        if tag == 1:
            monkeypatch.delenv("DMGS_TAIL_SPINS")
        else:
            reqs[tag] = (P, c, t, "vjp")
        batch.add(B, P, c, t, "vjp", tag)
    done = B.run()
    assert [d["status"] for d in done if d["tag"] == 1] == [_abi.DMGS_ERR_NONFINITE]
    batch.check_against_solo(reqs, [d for d in done if d["tag"] != 1])
