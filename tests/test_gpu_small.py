"""The single-workgroup coarse kernel against the oracle's fixed-cycle maps.

Grids whose coarse end begins at each shape the kernel takes: one exactly
solved level (N = 4, 6), a first level of 6 or 8 cells (12, 16), of 12 and 16
cells (24, 32, the latter with four levels), with no pre- or no
post-smoothing, in both cycle orders and face means; in two dimensions first
levels of 4 to 64 cells (128: six levels) and block passes on one tile, on
several with a ragged last one, and at the edge of the grid.

Tolerances: float64 1e-12 of the largest entry, as every fixed-cycle
comparison (rounding order over tens of stencil applications).  Float32
cycles inside refinement: a correction is formed in float32 and agrees to
2e-5 per pass as the float32 passes do; three steps of at most four levels
give 3 * 4 * 2e-5 = 2.4e-4 of the largest entry, against the iterate of as
many float64 cycles.
"""
import numpy as np
import pytest

from gpu_util import dev, host, rel_max, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [4, 6, 12, 16, 24, 32])
@pytest.mark.parametrize("nu", [(2, 2), (0, 2), (2, 0), (1, 3)])
@pytest.mark.parametrize("face_mean", ["arith", "harmonic"])
def test_small_levels_fp64(N, nu, face_mean):
    from oracle import ref
    from paper_2608_00760_amd import synth
    from paper_2608_00760_amd.solver import Options, Plan
    say("small levels fp64 N=%d nu=%s %s" % (N, nu, face_mean))
    c = synth.grf_case(N, 700 + N)
    H = ref.Hierarchy(c["D"], c["mua"], face_mean=face_mean)
    P = Plan(Options(N, fixed_cycles=3, nu_pre=nu[0], nu_post=nu[1], face_mean=face_mean))
    P.set_coefficients(dev(c["D"]), dev(c["mua"]))
    rho, _ = P.forward(dev(c["q"]))
    rr, _ = H.forward(c["q"], fixed_cycles=3, nu1=nu[0], nu2=nu[1])
    assert rel_max(host(rho), rr) <= 1e-12
    (qb, _, _), _ = P.vjp(rho, dev(c["rhobar"]))
    (rqb, _, _), _ = H.vjp(rr, c["rhobar"], fixed_cycles=3, nu1=nu[0], nu2=nu[1])
    assert rel_max(host(qb), rqb) <= 1e-12
    P.close()


@pytest.mark.parametrize("N", [4, 12, 24, 32])
@pytest.mark.parametrize("face_mean", ["arith", "harmonic"])
def test_small_levels_fp32(N, face_mean):
    from oracle import ref
    from paper_2608_00760_amd import synth
    from paper_2608_00760_amd.solver import Options, Plan
    say("small levels fp32 N=%d %s" % (N, face_mean))
    c = synth.grf_case(N, 800 + N)
    H = ref.Hierarchy(c["D"], c["mua"], face_mean=face_mean)
    P = Plan(Options(N, precision="fp32-in-fp64", fixed_cycles=3, ir_inner_cycles=1, face_mean=face_mean))
    P.set_coefficients(dev(c["D"]), dev(c["mua"]))
    rho, _ = P.forward(dev(c["q"]))
    assert rel_max(host(rho), H.forward(c["q"], fixed_cycles=3)[0]) <= 2.4e-4
    (qb, _, _), _ = P.vjp(rho, dev(c["rhobar"]))
    assert rel_max(host(qb), H.vjp(host(rho), c["rhobar"], fixed_cycles=3)[0][0]) <= 2.4e-4
    P.close()


@pytest.mark.parametrize("N,nu", [(8, (2, 2)), (12, (0, 2)), (24, (2, 0)), (48, (1, 3)), (64, (2, 2)), (96, (2, 0)),
                                  (128, (2, 2)), (192, (2, 2)), (384, (2, 2))])
@pytest.mark.parametrize("face_mean,g", [("arith", 0.0), ("harmonic", 0.4)])
def test_small_levels_and_blocks_2d(N, nu, face_mean, g):
    from oracle import ref2d
    from paper_2608_00760_amd import synth
    from paper_2608_00760_amd.solver import Options, Plan
    say("small levels 2d N=%d nu=%s %s" % (N, nu, face_mean))
    c = synth.grf_case(N, 900 + N, ndim=2)
    H = ref2d.Hierarchy2D(c["D"], c["mua"], face_mean=face_mean, g=g)
    P = Plan(Options(N, ndim=2, fixed_cycles=3, nu_pre=nu[0], nu_post=nu[1], face_mean=face_mean, bc_value=g))
    P.set_coefficients(dev(c["D"]), dev(c["mua"]))
    rho, _ = P.forward(dev(c["q"]))
    assert rel_max(host(rho), H.forward(c["q"], fixed_cycles=3, nu1=nu[0], nu2=nu[1])[0]) <= 1e-12
    (qb, _, _), _ = P.vjp(rho, dev(c["rhobar"]))
    rqb = H.vjp(host(rho), c["rhobar"], fixed_cycles=3, nu1=nu[0], nu2=nu[1])[0][0]
    assert rel_max(host(qb), rqb) <= 1e-12
    P.close()
