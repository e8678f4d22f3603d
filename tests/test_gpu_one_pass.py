"""GPU: the one-pass form of the general kernel (long single-period slices, rows read once per
iteration from tiles in device memory), reached here with explicit grids whose slices of
the rows exceed LDS, at the edges of its tiles (16 rows; 8 and 16 assets; four waves).

FP64: the weights of two kernels that run the same iteration differ by rounding only (about
1e-16 per iteration, a few thousand iterations), so 1e-10 of the largest weight, against
the default call.  FP32: the rows are floats and the iterates float offsets, so each weight
is known to about 1e-7 of the largest one; both FP32 forms end within the tolerance of the
same problem, whose objective is flat to first order: the oracle's relative KKT at twice the
tolerance, and objectives within it."""
import numpy as np
import pytest

from oracle.problem import kkt, normalize
from synth import make_single

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = 1e-6


def _solve(inst, **kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_22625_amd as ff
    print(f"[case] n={inst['n']} k={inst['k']} m={inst['m']} d={inst['d']} {kw}", flush=True)
    r = ff.solve_instance(inst, **{**dict(tol=TOL, time_limit_s=20.0, max_iter=100_000, return_dual=True,
                                          raise_on_failure=False), **kw})
    torch.cuda.synchronize()
    return r


def _kkt(inst, W, Y):
    pb = normalize(inst, factor=np.linalg.cholesky(inst["Omega"]) if inst["k"] else np.zeros((0, 0)))
    return kkt(pb, W.cpu().numpy(), *(y.cpu().numpy() for y in Y)).rel_kkt


@pytest.mark.parametrize("n,k,m,wg,d", [
    (1400, 10, 6, 1, 1.5), (1501, 9, 5, 1, 2.0), (1409, 10, 7, 1, 1.5),       # 16, 14 and 17 rows
    (1711, 24, 24, 3, 1.5), (1300, 24, 25, 2, 1.5),                          # 48 and 49 rows
    (1215, 40, 40, 4, 2.0), (1216, 41, 40, 3, 1.5), (1217, 56, 56, 5, 1.5),  # 80, 81 and 112 rows
    (1030, 60, 80, 5, 1.5), (1033, 64, 81, 6, 1.5), (1100, 80, 80, 6, 1.5)]) # 140, 145 and 160 rows
def test_fp64_matches_the_default_call(n, k, m, wg, d):
    assert (k + m) * -(-n // wg) * 8 > 160 * 1024      # the slice of the rows exceeds LDS
    inst = make_single(n, k, m, seed=n + m, d=d)
    (W, i, Y), (Wd, di, Yd) = _solve(inst, workgroups=wg), _solve(inst)
    assert i.status == 0 and di.status == 0 and i.iters == di.iters
    assert float((W - Wd).abs().max()) <= 1e-10 * float(Wd.abs().max())
    assert _kkt(inst, W, Y) <= 2.0 * TOL


@pytest.mark.parametrize("n,k,m,wg", [(2801, 10, 6, 1), (1310, 20, 44, 2), (1537, 60, 80, 5), (1290, 60, 88, 4)])
def test_fp32_reaches_the_tolerance(n, k, m, wg):
    assert (k + m) * -(-n // wg) * 4 > 160 * 1024
    inst = make_single(n, k, m, seed=n)
    (W, i, Y), (Wd, di, Yd) = _solve(inst, workgroups=wg, precision="fp32"), _solve(inst)
    assert i.status == 0 and di.status == 0
    assert _kkt(inst, W, Y) <= 2.0 * TOL
    assert abs(i.primal_obj - di.primal_obj) <= 2.0 * TOL * abs(di.primal_obj)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_warm_start_cut_off_and_deterministic(precision):
    inst = make_single(2100, 40, 40, seed=3)
    inst["U"][0], inst["L"][1] = np.inf, -np.inf
    kw = dict(workgroups=1, precision=precision)
    W, i, Y = _solve(inst, max_iter=200, **kw)
    assert i.status == 4 and i.iters == 200
    W, i, Y = _solve(inst, w_init=W, y_init=Y, omega_init=i.omega, **kw)
    assert i.status == 0 and _kkt(inst, W, Y) <= 2.0 * TOL
    a, b = (_solve(inst, deterministic=True, workgroups=3, precision=precision) for _ in range(2))
    assert a[1].status == 0 and torch.equal(a[0], b[0])
