"""2D FP64 of degree 6 to 8: plain 1D products on few blocks, even-odd ones on
many.  The rule counts blocks over all right-hand sides, so the first column of
two calls that differ by one column, just below and just above the line, goes
both ways."""
import numpy as np
import pytest

import synth
from tests.gpu_common import log, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("gl", [0, 1])
@pytest.mark.parametrize("p,cols", [(6, 20), (7, 17), (8, 7)])
def test_plain_equals_even_odd(p, cols, gl):
    import paper_2510_00998_amd as hp
    n = 30
    cpb = 256 // (p + 1)
    blocks, line = -(-n * n // cpb), 256 if p == 8 else 512
    assert blocks * cols <= line < blocks * (cols + 1)
    s = hp.Solver(2, n, p, 1.3, max_rhs=cols + 1, basis=gl)
    u = synth.random_vector((cols + 1) * s.ndof, seed=71 + p)
    b = synth.random_rhs((cols + 1) * s.ndof, seed=72 + p)
    got = []
    for k in (cols, cols + 1):
        log(f"plain 2D p={p} gl={gl} columns {k}")
        ud, bd = to_dev(u[:k * s.ndof], torch.float64), to_dev(b[:k * s.ndof], torch.float64)
        y = s.apply_A(ud, torch.empty_like(ud), nrhs=k)
        v = s.smooth(ud.clone(), bd, 2, nrhs=k)
        w = s.vcycle(ud.clone(), bd, nrhs=k)
        got.append([to_host(x)[:s.ndof] for x in (y, v, w)])
    # both sum the same products in another order: 1e-12 for one apply, 1e-11
    # for the sweeps and the cycle, as the parity with the oracle
    for x, r, tol in zip(got[0], got[1], (1e-12, 1e-11, 1e-11)):
        assert np.isfinite(x).all()
        assert rel_err(x, r) <= tol
