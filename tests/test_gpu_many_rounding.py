"""GPU: a market's FP32 result in ffo_solve_many does not depend on the other markets of the call.
A market of one workgroup sums in a fixed order, so its weights are the same bits."""
import pytest

from synth import make_single

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("others", [12, 60])
def test_neighbours_do_not_change_a_result(others):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_22625_amd as ff
    small, big = make_single(200, 60, 80, seed=1), make_single(5000, 60, 80, seed=2)
    print(f"[case] many FP32 beside {others}", flush=True)
    kw = dict(precision="fp32", max_iter=192, raise_on_failure=False)
    a, _ = ff.solve_many([small, big], **kw)
    b, _ = ff.solve_many([small] + [big] * others, **kw)
    assert torch.equal(a[0], b[0])
