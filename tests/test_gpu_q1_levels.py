"""Q1 levels of the V-cycle, in tiles and in one workgroup, at mesh sizes
around the tile edges: whole and ragged last tiles, coarse grids whose last
cell is smaller, both coarsening factors, every smoothing count the tiles take
and one they do not, two right-hand sides at once."""
import pytest

import synth
from oracle import Hierarchy, HierarchyOptions
from tests.gpu_common import log, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# one V-cycle of degree 1 or 2: some 20 smoothing steps and residuals in
# sequence, each good to about 10 u64 times the condition of the smoother
# (below 50): 1e-11 in FP64; FP32 as for the other V-cycle parity cases
TOL = {torch.float64: 1e-11, torch.float32: 1e-5}


@pytest.mark.parametrize("pre,post", [(1, 1), (2, 1), (1, 2), (2, 2), (3, 1), (0, 2)])
@pytest.mark.parametrize("dim,n,hf", [(2, 9, 2), (2, 24, 2), (2, 34, 2), (2, 51, 2), (2, 25, 3), (2, 39, 3),
                                      (3, 8, 2), (3, 10, 2), (3, 11, 2), (3, 19, 2), (3, 10, 3), (3, 14, 3)])
def test_q1_levels(dim, n, hf, pre, post):
    log(f"Q1 levels dim={dim} n={n} factor {hf} nu=({pre}, {post})")
    kw = dict(nu_pre_cg=pre, nu_post_cg=post, h_factor=hf)
    kappa = synth.kappa_log_uniform(dim, n, seed=61) if n % 2 else 1.3
    p = 2 if dim == 2 else 1
    H = Hierarchy(dim, n, p, kappa, opts=HierarchyOptions(**kw))
    nd = H.fine.ndof
    u0 = synth.random_vector(2 * nd, seed=62)
    b = synth.random_rhs(2 * nd, seed=63)
    ref = [H.vcycle(0, u0[c * nd:(c + 1) * nd].copy(), b[c * nd:(c + 1) * nd]) for c in range(2)]
    import paper_2510_00998_amd as hp
    g = hp.Solver(dim, n, p, kappa, max_rhs=2, **kw)
    for dt, tol in TOL.items():
        ud, bd = to_dev(u0, dt), to_dev(b, dt)
        g.vcycle(ud, bd, nrhs=2)
        got = to_host(ud)
        for c in range(2):
            err = rel_err(got[c * nd:(c + 1) * nd], ref[c])
            log(f"  {dt} column {c}: rel err {err:.3e}")
            assert err <= tol


@pytest.mark.parametrize("pre,post", [(1, 2), (2, 2), (3, 1)])
def test_q1_levels_of_a_batch(pre, post):
    """maxit = 1 from u0 = 0: u1 = alpha z, z = V-cycle(r0), problems without,
    with one and with two tiled Q1 levels and with one Q1 level in all."""
    import paper_2510_00998_amd as hp
    problems = [(2, 1), (4, 2), (9, 3), (10, 1), (13, 2), (19, 1)]
    log(f"Q1 levels of a batch nu=({pre}, {post})")
    kw = dict(nu_pre_cg=pre, nu_post_cg=post)
    solvers = [hp.Solver(3, n, p, 1.7, max_rhs=2, **kw) for n, p in problems]
    batch = hp.Batch(solvers)
    us, bs, refs = [], [], []
    for (n, p), s in zip(problems, solvers):
        H = Hierarchy(3, n, p, 1.7, opts=HierarchyOptions(**kw))
        A, nd = H.levels[0].A, s.ndof
        b = synth.random_rhs(2 * nd, seed=64 + n)
        ref = []
        for r in range(2):
            br = b[r * nd:(r + 1) * nd]
            z = H.precondition(br)
            ref.append((z @ br) / (z @ (A @ z)) * z)
        refs.append(ref)
        us.append(torch.zeros(2 * nd, dtype=torch.float64, device="cuda"))
        bs.append(to_dev(b, torch.float64))
    _, st = batch.solve(us, bs, rtol=1e-14, maxit=1, nrhs=2, check=False)
    assert st == 4  # not converged after one iteration
    for (n, p), s, u, ref in zip(problems, solvers, us, refs):
        got, nd = to_host(u), s.ndof
        for r in range(2):
            err = rel_err(got[r * nd:(r + 1) * nd], ref[r])
            log(f"  n={n} p={p} rhs={r}: rel err {err:.3e}")
            assert err <= TOL[torch.float32]
