"""GPU: the single-period kernel that holds the constraint rows in registers, at the edges
of its tiles (assets per workgroup and wave, groups of 16 rows, one and many workgroups),
against the oracle's KKT evaluation of the returned pair and the general kernel.

Tolerances: the oracle's relative KKT at twice the solver's tolerance (it evaluates the same
definition in another summation order); the weights of two kernels that run the same
iteration differ by rounding only (about 1e-16 per iteration, a few thousand iterations,
divisions replaced by reciprocals within 1 ulp), so 1e-10 of the largest weight."""
import numpy as np
import pytest

from oracle.problem import kkt, normalize
from synth import make_batch, make_single

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = 1e-7


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_22625_amd as ff
    return ff


def _both(inst, **kw):
    """The default call (rows in registers) and the general kernel (an explicit grid)."""
    ff = _gpu()
    n = inst["n"]
    print(f"[case] n={n} k={inst['k']} m={inst['m']} d={inst['d']} {kw}", flush=True)
    kw = {**dict(tol=TOL, time_limit_s=20.0, max_iter=100_000, return_dual=True, raise_on_failure=False), **kw}
    a = ff.solve_instance(inst, **kw)
    torch.cuda.synchronize()
    b = ff.solve_instance(inst, workgroups=max(1, min(200, n // 32)), **kw)
    torch.cuda.synchronize()
    return a, b


def _agree(inst, a, b):
    (W, i, Y), (Wg, ig, Yg) = a, b
    assert i.status == 0 and ig.status == 0 and i.iters == ig.iters
    assert float((W - Wg).abs().max()) <= 1e-10 * float(Wg.abs().max())
    pb = normalize(inst, factor=np.linalg.cholesky(inst["Omega"]) if inst["k"] else np.zeros((0, 0)))
    K = kkt(pb, W.cpu().numpy(), *(y.cpu().numpy() for y in Y))
    assert K.rel_kkt <= 2.0 * TOL, K


@pytest.mark.parametrize("n,k,m", [
    (1, 2, 1), (3, 0, 2), (17, 3, 13), (128, 10, 6), (129, 10, 7),       # one workgroup, 16 and 17 rows
    (256, 8, 24), (257, 8, 25), (512, 20, 12), (513, 20, 12),            # 32 and 33 rows, one and two workgroups
    (1025, 28, 20), (700, 40, 40), (700, 41, 40),                        # 48, 80 and 81 rows
    (1500, 60, 52), (1100, 60, 53), (2111, 64, 80), (900, 80, 80),       # 112, 113, 144 and 160 rows
    (11000, 6, 16), (5500, 60, 80)])                                     # two and more slot copies
def test_tile_edges(n, k, m):
    inst = make_single(n, k, m, seed=n + m)
    _agree(inst, *_both(inst))


@pytest.mark.parametrize("n,k,m", [(300, 10, 8), (1300, 30, 20)])
def test_quadratic_impact(n, k, m):
    inst = make_single(n, k, m, seed=n, d=2.0)
    _agree(inst, *_both(inst))


def test_more_rows_than_registers_hold_take_the_general_kernel():
    inst = make_single(400, 81, 80, seed=5)
    _agree(inst, *_both(inst))


@pytest.mark.parametrize("n", [200, 1200])
def test_warm_start_one_sided_bounds_and_cut_off(n):
    """Infinite bound sides, a warm start from a cut-off solve, and the iterate returned at
    an iteration limit that is not a multiple of the check interval."""
    inst = make_single(n, 12, 9, seed=n)
    inst["U"][0], inst["L"][1] = np.inf, -np.inf
    (W, i, Y), (Wg, ig, Yg) = _both(inst, max_iter=100)
    assert i.status == ig.status == 4 and i.iters == ig.iters == 100
    assert float((W - Wg).abs().max()) <= 1e-10 * float(Wg.abs().max())
    for y, yg in zip(Y, Yg):
        assert float((y - yg).abs().max()) <= 1e-10 * max(1e-3, float(yg.abs().max()))
    _agree(inst, *_both(inst, w_init=W, y_init=Y, omega_init=i.omega))


def test_many_markets_share_the_queue():
    """More workgroups than compute units, sizes from one asset to several workgroups: the
    tickets run in several waves and every market gets its own solve's result."""
    ff = _gpu()
    insts = [make_single(n, 6, 11, seed=100 + j) for j, n in enumerate([1, 5, 4000, 700, 513, 512, 129] * 20)]
    print(f"[case] many {len(insts)}", flush=True)
    Ws, infos = ff.solve_many(insts, tol=TOL, time_limit_s=20.0, max_iter=100_000)
    torch.cuda.synchronize()
    for j in (0, 1, 2, 3, 4, 5, 6, 72, len(insts) - 1):
        W, i = ff.solve_instance(insts[j], tol=TOL, time_limit_s=20.0, max_iter=100_000)
        assert infos[j].status == 0 and infos[j].iters == i.iters
        assert float((W - Ws[j]).abs().max()) <= 1e-10 * float(W.abs().max())


@pytest.mark.parametrize("B,cut", [(4, 100_000), (5, 100_000), (12, 100_000), (12, 700), (12, 1000)])
def test_default_batch_keeps_the_lockstep_results(B, cut):
    """The default batched form against the lockstep form asked for by name: the same
    iterations, restarts and statuses (the hand-off of the last instances and the iteration
    limit at a check included), the weights within rounding."""
    ff = _gpu()
    batch = make_batch(B, 10, 8, seed=B, n_lo=100, n_hi=900)
    print(f"[case] batch {B} {cut}", flush=True)
    kw = dict(tol=TOL, time_limit_s=20.0, max_iter=cut, raise_on_failure=False)
    W, a = ff.solve_batched(batch, **kw)
    Wl, b = ff.solve_batched(batch, form="lockstep", **kw)
    torch.cuda.synchronize()
    assert [(i.status, i.iters, i.restarts) for i in a] == [(i.status, i.iters, i.restarts) for i in b]
    assert float((W - Wl).abs().max()) <= 1e-10 * float(Wl.abs().max())
