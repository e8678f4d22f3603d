"""GPU: impact coefficients so large that their squares overflow (an asset that must not trade),
on the register kernels and the general kernel: the same iteration at a fixed number of
iterations, weights within 1e-10 of the largest."""
import numpy as np
import pytest

from synth import make_multi, make_single

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("q", [1e100, 1e160, 1e300])
@pytest.mark.parametrize("T,d", [(0, 1.5), (0, 2.0), (4, 1.5)])
def test_register_kernels_match_the_general_kernel(q, T, d):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_22625_amd as ff
    inst = make_multi(T, 300, 6, 5, seed=3, d=d) if T else make_single(300, 6, 5, seed=3, d=d)
    inst["q"] = np.array(inst["q"])
    inst["q"][..., ::7] = q
    print(f"[case] q={q} T={T} d={d}", flush=True)
    kw = dict(max_iter=128, time_limit_s=20.0, raise_on_failure=False)
    W, i = ff.solve_instance(inst, **kw)
    Wg, ig = ff.solve_instance(inst, workgroups=5, **kw)
    assert i.status == ig.status and i.iters == ig.iters
    assert bool(torch.isfinite(W).all())
    assert float((W - Wg).abs().max()) <= 1e-10 * float(Wg.abs().max())
