"""Block shapes of single-problem 3D traversals.  Constant kappa: runs of cells on
small meshes, bricks above, on the largest mesh of runs and on meshes just above
the line, with whole and ragged bricks along every axis, against an adaptive
mesh without refinement, which takes runs at every size.  Variable kappa: its
own bricks, on meshes with facets between bricks along every axis, against the
operator and the sweep applied cell by cell in FP64 torch."""
import numpy as np
import pytest

import synth
from tests.gpu_common import log, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# The same arithmetic up to the order of sums: FP64 as the parity of one apply /
# two sweeps with the oracle (1e-12, 1e-11), FP32 1e-5.
TOL = {torch.float64: (1e-12, 1e-11), torch.float32: (1e-5, 1e-5)}
# the largest n in runs, FP64 and FP32 (degree 6 in FP32 always)
LINE = {(1, 8): 23, (1, 4): 29, (2, 8): 17, (2, 4): 22, (3, 8): 13, (3, 4): 13, (4, 8): 14, (4, 4): 30,
        (5, 8): 24, (5, 4): 30, (6, 8): 11, (7, 8): 8, (7, 4): 8, (8, 8): 8, (8, 4): 13}


def _uniform_leaves(n):
    c = np.arange(n ** 3)
    return np.stack([0 * c, c % n, c // n % n, c // (n * n)], axis=1).astype(np.int32)


@pytest.mark.parametrize("step", [0, 1, 2])
@pytest.mark.parametrize("p,size", sorted(LINE))
def test_shapes_agree_around_the_line(p, size, step):
    dt = {8: torch.float64, 4: torch.float32}[size]
    n = LINE[p, size] + step
    log(f"block shapes p={p} {dt} n={n}")
    import paper_2510_00998_amd as hp
    a = hp.Solver(3, n, p, 1.3)
    r = hp.Solver(3, n, p, 1.3, leaves=_uniform_leaves(n))
    ud = to_dev(synth.random_vector(a.ndof, seed=80 + p), dt)
    bd = to_dev(synth.random_rhs(a.ndof, seed=81 + p), dt)
    ya = a.apply_A(ud, torch.empty_like(ud))
    yr = r.apply_A(ud, torch.empty_like(ud))
    err = float((ya - yr).abs().max() / yr.abs().max())
    log(f"  apply {err:.2e}")
    assert err <= TOL[dt][0]
    ua, ur = ud.clone(), ud.clone()
    a.project(ua)
    a.sweep(ua, bd, 2)
    r.smooth(ur, bd, 2)
    err = float((ua - ur).abs().max() / ur.abs().max())
    log(f"  sweeps {err:.2e}")
    assert err <= TOL[dt][1]


@pytest.mark.parametrize("p,n", [(1, 5), (1, 9), (2, 4), (2, 7), (3, 5), (3, 7), (4, 6), (4, 7), (5, 4), (5, 7), (6, 6),
                                 (6, 7), (7, 3), (7, 5), (8, 4), (8, 5)])
def test_variable_kappa_bricks(p, n):
    from perf.cases import _Cells
    import paper_2510_00998_amd as hp
    log(f"variable kappa bricks p={p} n={n}")
    kappa = synth.kappa_log_uniform(3, n, seed=82 + p)
    ref = _Cells(n, p, kappa)
    s = hp.Solver(3, n, p, kappa)
    for dt, (tol_apply, tol_smooth) in TOL.items():
        ud = to_dev(synth.random_vector(s.ndof, seed=83 + p), dt)
        bd = to_dev(synth.random_rhs(s.ndof, seed=84 + p), dt)
        shape = (n,) * 3 + (p + 1,) * 3
        y = s.apply_A(ud, torch.empty_like(ud))
        err = rel_err(to_host(y), ref.apply(ud.double().reshape(shape)).reshape(-1).cpu().numpy())
        log(f"  {dt} apply {err:.2e}")
        assert err <= tol_apply
        want = ref.smooth(ud.double(), bd.double(), 2).cpu().numpy()
        err = rel_err(to_host(s.smooth(ud.clone(), bd, 2)), want)
        log(f"  {dt} sweeps {err:.2e}")
        assert err <= tol_smooth
