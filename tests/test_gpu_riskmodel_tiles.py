"""GPU: the one-launch risk model at the edges of its tiles (16 assets, steps of 128 days,
chunks of 512 days of factor returns) and for every factor count, against the oracle's
plain least squares.  Tolerances: sums of at most 1,200 terms in another order and a
normal-equation solve of a well-conditioned Gram matrix (condition below 1e4), so about
1,200 * 1e-16 * 1e4 ~ 1e-9 relative at the worst."""
import numpy as np
import pytest

from oracle.riskmodel import risk_model as oracle_risk_model

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _panel(days, n, p, seed, masked):
    rng = np.random.default_rng(seed)
    Fr = rng.standard_normal((days, p)) * 0.01
    R = Fr @ rng.standard_normal((p, n)) + rng.standard_normal((days, n)) * 0.02
    M = None
    if masked:
        M = (rng.random((days, n)) > 0.1).astype(np.uint8)
        M[: days // 2, :: 5] = 0
        M[:, n - 1] = 0              # never observed
    return R, Fr, M


@pytest.mark.parametrize("days,n,p,masked", [
    (127, 15, 1, False), (128, 16, 2, True), (129, 17, 3, False), (511, 33, 4, True), (512, 129, 5, False),
    (513, 64, 6, True), (640, 300, 7, False), (1025, 47, 8, True), (1152, 1, 8, False), (60, 2100, 6, True)])
def test_tile_edges(days, n, p, masked):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_22625_amd as ff
    R, Fr, M = _panel(days, n, p, days + n, masked)
    print(f"[case] risk days={days} n={n} p={p} masked={masked}", flush=True)
    seen = R if M is None else np.where(M == 0, np.nan, R)     # unobserved entries do not count, whatever they hold
    beta, Sf, D, valid = ff.risk_model(seen, Fr, mask=M, min_obs=min(42, days))
    torch.cuda.synchronize()
    ref = oracle_risk_model(R, Fr, mask=M, min_obs=min(42, days))
    np.testing.assert_array_equal(valid.cpu().numpy().astype(bool), ref.valid)
    np.testing.assert_allclose(beta.cpu().numpy(), ref.beta, rtol=1e-9, atol=1e-9)
    np.testing.assert_allclose(D.cpu().numpy(), ref.D, rtol=1e-9, atol=1e-20)
    np.testing.assert_allclose(Sf.cpu().numpy(), ref.Sigma_f, rtol=1e-12, atol=1e-17)
