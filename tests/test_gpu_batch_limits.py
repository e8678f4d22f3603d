"""GPU: the limits of a batched call.  The default form's time limit is the call's, as in the
lockstep form it stands in for, whatever the number of instances that wait for a compute unit,
and an instance that converged within max_iter stays converged."""
import pytest

from synth import make_batch, make_single

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TIMEOUT = 7


def _ff():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_22625_amd as ff
    return ff


@pytest.mark.parametrize("form,check_every", [("auto", 64), ("auto", 4), ("lockstep", 64)])
def test_time_limit_covers_the_call(form, check_every):
    """600 one-workgroup instances (more than twice the compute units) that run on until their
    error is zero to the last bit, which few reach in time.  Past the limit each runs to its next check at most, a few milliseconds in all: half of the
    limit again is allowed for that and the clocks."""
    ff = _ff()
    batch = make_batch(600, 4, 6, seed=41, n_lo=40, n_hi=400)
    limit = 0.2
    print(f"[case] time limit {form} check_every={check_every}", flush=True)
    W, infos = ff.solve_batched(batch, form=form, tol=1e-30, check_every=check_every, max_iter=10**9,
                                time_limit_s=limit, raise_on_failure=False)
    print(f"[case] {infos[0].ms_iter:.1f} ms", flush=True)
    assert infos[0].ms_iter <= 1.5e3 * limit, infos[0].ms_iter
    assert {i.status for i in infos} in ({TIMEOUT}, {0, TIMEOUT})
    assert bool(torch.isfinite(W).all())


def test_every_market_of_a_call_has_the_limit():
    """ffo_solve_many and the team form count the limit for each instance: those that wait for a
    compute unit get it too (5 us an iteration and one workgroup here, at most three of them waiting
    in turn)."""
    ff = _ff()
    limit = 0.05
    print("[case] time limit many", flush=True)
    _, a = ff.solve_many([make_single(40 + j % 60, 4, 6, seed=j) for j in range(300)], tol=1e-30, max_iter=10**9,
                         time_limit_s=limit, raise_on_failure=False)
    _, b = ff.solve_batched(make_batch(600, 4, 6, seed=41, n_lo=40, n_hi=400), form="teams", tol=1e-30, max_iter=10**9,
                            time_limit_s=limit, raise_on_failure=False)
    for infos, waves in ((a, 2), (b, 3)):
        late = [i.iters for i in infos if i.status == TIMEOUT]
        assert late and min(late) * 10e-6 >= 0.5 * limit
        assert infos[0].ms_iter <= 1.5e3 * limit * waves


def test_instances_that_converged_in_time_keep_their_results():
    ff = _ff()
    batch = make_batch(600, 4, 6, seed=43, n_lo=40, n_hi=400)
    kw = dict(tol=1e-7, max_iter=100_000, raise_on_failure=False)
    print("[case] time limit half-way", flush=True)
    W, a = ff.solve_batched(batch, time_limit_s=30.0, **kw)
    limit = 0.5e-3 * a[0].ms_iter
    Wc, b = ff.solve_batched(batch, time_limit_s=limit, **kw)
    done = [j for j, i in enumerate(b) if i.status == 0]
    assert all(i.status == 0 for i in a) and {i.status for i in b} == {0, TIMEOUT}
    assert b[0].ms_iter <= 1.5e3 * limit + 10.0      # (at least one check interval of the instances that waited)
    handed = sorted((i.iters for i in a), reverse=True)[4]
    for j in done:
        if a[j].iters > handed:       # (continued from the hand-off there, not here)
            continue
        o, e = int(batch["offs"][j]), int(batch["offs"][j + 1])
        assert b[j].iters == a[j].iters and float((Wc[o:e] - W[o:e]).abs().max()) <= 1e-10 * float(W[o:e].abs().max())


@pytest.mark.parametrize("check_every,seed,j", [(64, 19, 0), (4, 14, 3)])   # iterates kept, and a second run
def test_hand_off_keeps_a_converged_result(check_every, seed, j):
    """Instance j, of the four that a hand-off continues, takes more iterations from there than its
    team did: with the team's count as the limit the team's result is the answer."""
    ff = _ff()
    batch = make_batch(6, 6, 5, seed=seed, n_lo=40, n_hi=400)
    print(f"[case] converged hand-off check_every={check_every}", flush=True)
    kw = dict(tol=1e-7, check_every=check_every, time_limit_s=20.0, raise_on_failure=False)
    Wt, t = ff.solve_batched(batch, form="teams", max_iter=100_000, **kw)
    cut = t[j].iters
    W, a = ff.solve_batched(batch, max_iter=cut, **kw)
    assert ff.solve_batched(batch, max_iter=100_000, **kw)[1][j].iters > cut
    for b, (i, it) in enumerate(zip(a, t)):     # (a hand-off may also converge earlier than the team)
        assert i.status == 0 or it.iters > cut, (b, i)
    o, e = int(batch["offs"][j]), int(batch["offs"][j + 1])
    assert a[j].iters == cut and a[j].rel_kkt <= 1e-7
    assert float((W[o:e] - Wt[o:e]).abs().max()) <= 1e-10 * float(Wt[o:e].abs().max())
