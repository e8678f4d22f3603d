"""GPU: the hand-off of the default batched form's last instances, from the iterates kept at the
checks and, where the longest ran too many checks past it, from a second run, against the
lockstep form.  Both run the same iterations, in another summation order (about 1e-16 per
iteration, a few thousand of them): weights within 1e-10 of the largest."""
import pytest

from synth import make_batch

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("check_every", [64, 4])   # a few checks past the hand-off, and hundreds
def test_hand_off_matches_the_lockstep_form(check_every):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_22625_amd as ff
    batch = make_batch(12, 10, 8, seed=12, n_lo=100, n_hi=900)
    print(f"[case] batch hand-off check_every={check_every}", flush=True)
    kw = dict(tol=1e-7, check_every=check_every, time_limit_s=30.0, max_iter=100_000, raise_on_failure=False)
    W, a = ff.solve_batched(batch, **kw)
    Wl, b = ff.solve_batched(batch, form="lockstep", **kw)
    its = sorted((i.iters for i in a), reverse=True)
    assert [i.iters for i in a] == [i.iters for i in b] and all(i.status == 0 for i in a)
    if check_every == 4:
        assert its[0] - its[4] > 32 * check_every      # more checks than are kept
    assert float((W - Wl).abs().max()) <= 1e-10 * float(Wl.abs().max())
