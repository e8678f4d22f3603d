"""GPU: the multi-period kernel that holds the constraint rows in registers, at the edges of
its tiles (periods per wave, tiles of 16 periods and 16 rows, 64 assets per workgroup), against
the oracle's KKT evaluation of the returned pair and the general kernel.

Tolerances as in test_gpu_row_registers.py: the oracle's relative KKT at twice the solver's
tolerance; the weights of two kernels that run the same iteration within 1e-10 of the largest."""
import numpy as np
import pytest

from oracle.problem import kkt, normalize
from synth import make_multi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = 1e-6


def _both(inst, **kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_22625_amd as ff
    n = inst["n"]
    print(f"[case] n={n} T={inst['T']} k={inst['k']} m={inst['m']} d={inst['d']} {kw}", flush=True)
    kw = {**dict(tol=TOL, time_limit_s=20.0, max_iter=100_000, return_dual=True, raise_on_failure=False), **kw}
    a = ff.solve_instance(inst, **kw)
    torch.cuda.synchronize()
    b = ff.solve_instance(inst, workgroups=max(1, min(200, n // 24)), **kw)
    torch.cuda.synchronize()
    return a, b


def _agree(inst, a, b):
    (W, i, Y), (Wg, ig, Yg) = a, b
    assert i.status == 0 and ig.status == 0 and i.iters == ig.iters
    assert float((W - Wg).abs().max()) <= 1e-10 * float(Wg.abs().max())
    pb = normalize(inst, factor=np.linalg.cholesky(inst["Omega"]) if inst["k"] else np.zeros((0, 0)))
    K = kkt(pb, W.cpu().numpy(), *(y.cpu().numpy() for y in Y))
    assert K.rel_kkt <= 2.0 * TOL, K


@pytest.mark.parametrize("T,n,k,m", [
    (2, 70, 3, 5), (3, 1, 2, 1), (3, 63, 2, 5), (8, 64, 10, 22), (9, 65, 10, 23),      # 8 and 9 trades, 32 and 33 rows
    (16, 130, 8, 5), (17, 129, 8, 5),                                    # one and two tiles of periods
    (4, 200, 24, 24), (4, 200, 24, 25), (5, 333, 40, 40), (5, 333, 40, 41),   # 48, 49, 80 and 81 rows
    (24, 70, 12, 4), (25, 70, 12, 4), (31, 40, 4, 3), (32, 40, 4, 3),   # 24, 25 and 32 trades
    (6, 500, 56, 56), (3, 2700, 5, 6)])                                  # 112 rows; two slot copies
def test_tile_edges(T, n, k, m):
    inst = make_multi(T, n, k, m, seed=T + n + m)
    _agree(inst, *_both(inst))


@pytest.mark.parametrize("T,n,k,m", [(33, 40, 4, 3), (4, 150, 57, 56)])
def test_beyond_the_tiles_takes_the_general_kernel(T, n, k, m):
    inst = make_multi(T, n, k, m, seed=T + n)
    _agree(inst, *_both(inst))


def test_quadratic_impact_no_rows_and_an_inactive_budget():
    inst = make_multi(5, 150, 6, 7, seed=3, d=2.0)
    _agree(inst, *_both(inst))
    inst = make_multi(4, 90, 0, 0, seed=4)
    _agree(inst, *_both(inst))
    inst = make_multi(4, 150, 6, 7, seed=5, lambda1=1e-6)   # heavy risk: the budget's multiplier is zero
    _agree(inst, *_both(inst))


def test_warm_start_one_sided_bounds_and_cut_off():
    inst = make_multi(6, 180, 12, 9, seed=8)
    inst["U"][0], inst["L"][1] = np.inf, -np.inf
    (W, i, Y), (Wg, ig, Yg) = _both(inst, max_iter=100)
    assert i.status == ig.status == 4 and i.iters == ig.iters == 100
    assert float((W - Wg).abs().max()) <= 1e-10 * float(Wg.abs().max())
    for y, yg in zip(Y, Yg):
        assert float((y - yg).abs().max()) <= 1e-10 * max(1e-3, float(yg.abs().max()))
    _agree(inst, *_both(inst, w_init=W, y_init=Y, omega_init=i.omega))
