"""Nodal and dual form of the cell traversals at every degree, on meshes
whose waves hold no interior cell (n = 2), a mix (n = 3, 4) and, with the
interior-cell block, interior classes only."""
import numpy as np
import pytest

import synth
from oracle import SIPG, Hierarchy, HierarchyOptions
from tests.gpu_common import log, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# FP64: about 10 u64 per stage over at most 9 stages of N <= 9 terms, times
# the condition of Mhat (below 50 per axis at degree 8): 1e-12 for one apply,
# 1e-11 for two sweeps; FP32 by the ratio of the unit roundoffs of a
# well-conditioned sum, 1e-5 as for the other FP32 parity cases.
TOL = {torch.float64: (1e-12, 1e-11), torch.float32: (1e-5, 1e-5)}


@pytest.mark.parametrize("p", range(1, 9))
@pytest.mark.parametrize("n,kind", [(2, "const"), (4, "const"), (3, "var"), (3, "interior")])
def test_traversals_of_every_degree(p, n, kind):
    log(f"traversals 3D n={n} p={p} {kind}")
    kappa = synth.kappa_log_uniform(3, n, seed=41) if kind == "var" else 1.7
    block = "interior" if kind == "interior" else "exact"
    if kind == "var" or n <= 3 or p <= 5:  # the oracle's matrix stays small
        H = Hierarchy(3, n, p, kappa, HierarchyOptions(block=block))
        s = H.fine
    else:
        H, s = None, SIPG(3, n, p, kappa)
    import paper_2510_00998_amd as hp
    g = hp.Solver(3, n, p, kappa, block_variant=1 if kind == "interior" else 0)
    u = synth.random_vector(s.ndof, seed=42 + p)
    b = synth.random_rhs(s.ndof, seed=43 + p)
    y_ref = s.A @ u
    u_ref = H.smooth(0, u.copy(), b, 2) if H is not None else None
    for dt, (tol_apply, tol_smooth) in TOL.items():
        ud, bd = to_dev(u, dt), to_dev(b, dt)
        yd = torch.empty_like(ud)
        g.apply_A(ud, yd)
        err = rel_err(to_host(yd), s.A @ u.astype(np.float32).astype(np.float64) if dt == torch.float32 else y_ref)
        log(f"  {dt} apply {err:.2e}")
        assert err <= tol_apply
        if u_ref is not None:
            g.smooth(ud, bd, 2)
            err = rel_err(to_host(ud), u_ref)
            log(f"  {dt} smooth {err:.2e}")
            assert err <= tol_smooth
