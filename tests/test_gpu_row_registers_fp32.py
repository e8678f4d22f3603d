"""GPU: the FP32 form on the kernel that holds the constraint rows in registers, against the
general kernel's FP32 form, which rounds the same values at the same places.

Tolerances: both forms round each stored iterate to a float offset from its anchor (6e-8 of the
offset) and evaluate in FP64, in another order of sums, so a few of those roundings fall the
other way: at a fixed number of iterations within 1e-6 of the largest weight.  Converged, the
oracle's FP64 relative KKT is at most twice the solver's tolerance: the check reads the
unrounded rows."""
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
    print(f"[case] fp32 n={inst['n']} k={inst['k']} m={inst['m']} d={inst['d']} {kw}", flush=True)
    r = ff.solve_instance(inst, **{**dict(tol=TOL, time_limit_s=20.0, max_iter=100_000, return_dual=True,
                                          raise_on_failure=False, precision="fp32"), **kw})
    torch.cuda.synchronize()
    return r


@pytest.mark.parametrize("n,k,m,d", [
    (17, 3, 13, 1.5), (129, 10, 7, 2.0), (513, 20, 12, 1.5), (700, 40, 41, 1.5), (1500, 60, 53, 1.5),
    (900, 80, 80, 2.0), (5500, 60, 80, 1.5)])
def test_matches_the_general_kernel(n, k, m, d):
    inst = make_single(n, k, m, seed=n, d=d)
    wg = max(1, min(200, n // 32))
    a, b = _solve(inst, max_iter=192), _solve(inst, max_iter=192, workgroups=wg)
    assert a[1].iters == b[1].iters == 192
    assert float((a[0] - b[0]).abs().max()) <= 1e-6 * float(b[0].abs().max())
    W, i, Y = _solve(inst)
    assert i.status == 0
    pb = normalize(inst, factor=np.linalg.cholesky(inst["Omega"]))
    assert kkt(pb, W.cpu().numpy(), *(y.cpu().numpy() for y in Y)).rel_kkt <= 2.0 * TOL


def test_many_markets_and_a_warm_start():
    import paper_2604_22625_amd as ff
    insts = [make_single(n, 12, 9, seed=n) for n in (700, 41, 257, 90)]
    one = [_solve(i, max_iter=192) for i in insts]
    Ws, infos = ff.solve_many(insts, tol=TOL, max_iter=192, precision="fp32", raise_on_failure=False)
    for (W, i, _), Wm, im in zip(one, Ws, infos):
        assert im.iters == i.iters
        assert float((W - Wm.reshape(W.shape)).abs().max()) <= 1e-6 * float(W.abs().max())
    W, i, Y = one[0]
    W, i, Y = _solve(insts[0], w_init=W, y_init=Y, omega_init=i.omega)
    assert i.status == 0
