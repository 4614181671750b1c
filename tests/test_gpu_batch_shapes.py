"""Block shapes of the batched driver.  One mesh past the line of small meshes in
both types keeps the whole batch in bricks (full, half, all degrees in one
launch); without it the half bricks give way to runs of cells.  Every launch
configuration smooths alike, and as the problems smoothed one by one."""
import pytest

import synth
from tests.gpu_common import log, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SMALL = [(4, 1), (5, 4), (3, 5), (6, 3), (9, 2)]
ALL_TILES = sum(1 << (p + 1) for p in range(1, 6))
CONFIGS = [[512, 1] * 3 + [0] * 3, [700, 1] * 3 + [ALL_TILES] * 3, [300, 0] * 3 + [0] * 3,
           [1 << 30, 1] * 3 + [ALL_TILES] * 3, [1 << 30, 0] * 3 + [0] * 3]


@pytest.mark.parametrize("large", [False, True])
def test_every_shape_smooths_alike(large):
    import paper_2510_00998_amd as hp
    problems = SMALL + ([(23, 2)] if large else [])
    nrhs = 2
    solvers = [hp.Solver(3, n, p, 1.7, max_rhs=nrhs) for n, p in problems]
    batch = hp.Batch(solvers)
    u0 = [synth.random_vector(nrhs * s.ndof, seed=90 + j) for j, s in enumerate(solvers)]
    b0 = [synth.random_rhs(nrhs * s.ndof, seed=95 + j) for j, s in enumerate(solvers)]
    # the same per-cell arithmetic up to the order of sums: 1e-11 for three
    # sweeps in FP64, 1e-5 in FP32, as the parity of sweeps with the oracle
    for dt, tol in ((torch.float64, 1e-11), (torch.float32, 1e-5)):
        bs = [to_dev(b, dt) for b in b0]
        ref = []
        for s, u, b in zip(solvers, u0, bs):
            ref.append(to_host(s.smooth(to_dev(u, dt), b, 3, nrhs=nrhs)))
        batch.smooth([to_dev(u, dt) for u in u0], bs, 3, nrhs=nrhs)  # builds the plan
        for cfg in CONFIGS:
            log(f"batch shapes large={large} {dt} {cfg}")
            batch.set_tuning(cfg)
            us = [to_dev(u, dt) for u in u0]
            batch.smooth(us, bs, 3, nrhs=nrhs)
            for (n, p), u, r in zip(problems, us, ref):
                err = rel_err(to_host(u), r)
                assert err <= tol, (n, p, cfg, err)


def test_small_and_large_batches_solve():
    import paper_2510_00998_amd as hp
    for problems in (SMALL, SMALL + [(23, 2)]):
        solvers = [hp.Solver(3, n, p, 1.7) for n, p in problems]
        batch = hp.Batch(solvers)
        bs = [to_dev(synth.random_rhs(s.ndof, seed=99 + j), torch.float64) for j, s in enumerate(solvers)]
        us = [torch.zeros_like(b) for b in bs]
        batch.solve(us, bs, rtol=1e-10, maxit=100)
        for tiles in (0, ALL_TILES):
            batch.set_tuning([600, 1, 0, 0, 0, 0, tiles, 0, 0])
            vs = [torch.zeros_like(b) for b in bs]
            infos, st = batch.solve(vs, bs, rtol=1e-10, maxit=100)
            assert st == 0
            for s, u, v, b in zip(solvers, us, vs, bs):
                r = b - s.apply_A(v, torch.empty_like(v))
                res = float(r.norm() / b.norm())
                log(f"batch of {len(problems)}, tiles {tiles}: residual {res:.2e}")
                assert res <= 2e-10
                assert rel_err(to_host(v), to_host(u)) <= 1e-8
