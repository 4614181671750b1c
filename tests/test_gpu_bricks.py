"""Bricks of cells (3D uniform meshes) against runs of cells: the same mesh as
an adaptive one without refinement takes the kernels that work on runs and
read every trace from the buffers.  Mesh sizes below, at and just past the
brick's edge along every axis, one right-hand side and two."""
import numpy as np
import pytest

import synth
from tests.gpu_common import log, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# Both sides do the same arithmetic up to the order of sums: FP64 as the
# parity of one apply / two sweeps with the oracle (1e-12, 1e-11), FP32 1e-5.
TOL = {torch.float64: (1e-12, 1e-11), torch.float32: (1e-5, 1e-5)}


def _uniform_leaves(n):
    c = np.arange(n ** 3)
    return np.stack([0 * c, c % n, c // n % n, c // (n * n)], axis=1).astype(np.int32)


@pytest.mark.parametrize("p,n", [(1, 3), (1, 4), (1, 5), (1, 9), (2, 3), (2, 4), (2, 7), (3, 4), (3, 5), (3, 9),
                                 (4, 4), (4, 5), (4, 6), (4, 11), (5, 6), (5, 7), (5, 8), (6, 4), (6, 5), (6, 6),
                                 (7, 2), (7, 3), (7, 5), (8, 3), (8, 4)])
@pytest.mark.parametrize("nrhs", [1, 2])
def test_bricks_equal_runs(p, n, nrhs):
    log(f"bricks p={p} n={n} nrhs={nrhs}")
    import paper_2510_00998_amd as hp
    a = hp.Solver(3, n, p, 1.3, max_rhs=nrhs)
    r = hp.Solver(3, n, p, 1.3, max_rhs=nrhs, leaves=_uniform_leaves(n))
    assert a.ndof == r.ndof
    u = synth.random_vector(nrhs * a.ndof, seed=60 + p)
    b = synth.random_rhs(nrhs * a.ndof, seed=61 + p)
    for dt, (tol_apply, tol_smooth) in TOL.items():
        ud, bd = to_dev(u, dt), to_dev(b, dt)
        ya, yr = torch.empty_like(ud), torch.empty_like(ud)
        a.apply_A(ud, ya, nrhs=nrhs)
        r.apply_A(ud, yr, nrhs=nrhs)
        err = rel_err(to_host(ya), to_host(yr))
        log(f"  {dt} apply {err:.2e}")
        assert err <= tol_apply
        ua, ur = ud.clone(), ud.clone()
        a.project(ua, nrhs=nrhs)
        a.sweep(ua, bd, 2, nrhs=nrhs)
        r.smooth(ur, bd, 2, nrhs=nrhs)
        err = rel_err(to_host(ua), to_host(ur))
        log(f"  {dt} sweeps {err:.2e}")
        assert err <= tol_smooth
