"""Unrolled adjoint with the finest level in register blocks.

V(2,2) plans of at most 64 cells with a boundary value: the recorded phases
write interior vertices only, so the slots' boundary is the one they got when
they were allocated.  Both face means and both state policies against the
oracle (1e-12, as the other unrolled comparisons), twice on one plan with
other coefficients and inputs, so that reused slots are read too.
"""
import numpy as np
import pytest

from gpu_util import dev, host, rel_max, say
from test_gpu_unrolled import case, plan_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store", ["0", "1"])
@pytest.mark.parametrize("N,n", [(4, 2), (16, 3), (48, 2), (64, 2)])
@pytest.mark.parametrize("face_mean,g", [("arith", 0.4), ("harmonic", 0.3)])
def test_block_levels_with_a_boundary_value(N, n, face_mean, g, store, monkeypatch):
    from oracle import unrolled
    monkeypatch.setenv("DMGS_UNROLLED_STORE", store)
    say("unrolled blocks N=%d %s g=%g store=%s" % (N, face_mean, g, store))
    P = None
    for seed in (500 + N, 600 + N):
        logD, logmu, q, w = case(N, seed)
        if P is None:
            P = plan_for(N, logD, logmu, fixed_cycles=n, face_mean=face_mean, bc_value=g)
        else:
            P.set_log_coefficients(dev(logD), dev(logmu))
        (rho, (qb, gD, gmu)), _ = P.vjp_unrolled(dev(q), dev(w))
        U = unrolled.Unrolled(np.exp(logD), np.exp(logmu), g=g, harmonic=face_mean == "harmonic")
        rr, (rqb, rgD, rgmu) = U.vjp(q, w, n, 2, 2)
        errs = {name: rel_max(host(a), b) for name, a, b in (("rho", rho, rr), ("qbar", qb, rqb), ("logD", gD, rgD),
                                                             ("logmua", gmu, rgmu))}
        say("  errors", {k: "%.1e" % v for k, v in errs.items()})
        assert max(errs.values()) <= 1e-12, errs
    P.close()
