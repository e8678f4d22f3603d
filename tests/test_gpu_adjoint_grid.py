"""GPU: the adjoint kernel at the edges of its placement (rows and iteration arrays in LDS, rows
alone, neither) and of its grid (16 and 32 assets a workgroup, one workgroup, a last one with
few assets), against the adjoint of the same solution on another grid.

A fixed number of iterations: on these small degenerate markets the linear iteration need not
converge (a unit residual, on every grid).  Tolerance: 2,048 applications of the same linear
map in another summation order, about 1e-15 each, times the growth of the iterates against
the gradient, taken as at most 1e5: 2e-7 relative."""
import pytest

from synth import make_multi, make_single

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _gradients(inst, workgroups):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_22625_amd as ff
    kw = dict(tol=1e-8, max_iter=100_000, time_limit_s=20.0, return_dual=True)
    W, info, Y = ff.solve_instance(inst, **kw)
    g = torch.linspace(-1.0, 1.0, W.numel(), dtype=torch.float64, device=W.device).reshape(W.shape).contiguous()
    out = []
    for wg in workgroups:
        print(f"[case] adjoint n={inst['n']} T={inst['T']} rows={inst['k'] + inst['m']} workgroups={wg}", flush=True)
        orig = ff.default_options

        def options(wg=wg):
            o = orig()
            o.workgroups = wg
            return o
        ff.default_options = options
        try:
            out.append(ff.adjoint(inst, W, Y, g, omega=info.omega, max_iter=2048, time_limit_s=20.0, raise_on_failure=False))
        finally:
            ff.default_options = orig
        torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("T,n,k,m,other", [
    (0, 31, 4, 5, 3), (0, 33, 4, 5, 1), (4, 65, 5, 6, 2), (6, 15, 3, 4, 2),     # T >= 6: five periods and more
    (6, 17, 3, 4, 1), (8, 129, 10, 10, 3), (0, 2001, 10, 6, 30),
    (0, 700, 30, 30, 2), (0, 700, 30, 30, 1)])                                 # rows beside no arrays in LDS; neither
def test_grids_agree(T, n, k, m, other):
    inst = make_multi(T, n, k, m, seed=n + T) if T else make_single(n, k, m, seed=n)
    a, b = _gradients(inst, (0, other))
    assert a[3].iters == b[3].iters
    for x, y in zip(a[:3], b[:3]):
        assert float((x - y).norm()) <= 2e-7 * max(float(y.norm()), 1e-30)
