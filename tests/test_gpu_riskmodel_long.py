"""GPU: the risk model over long windows (512 threads a workgroup from 2048 days, up to 4096 assets;
steps of 128 days), against the oracle's plain least squares.  Tolerances: sums of 2,600 terms in
another order, an independent normal panel (condition of the Gram matrix below 10), so about
2,600 * 1e-16 * 10 = 3e-12; 1e-10 asked."""
import numpy as np
import pytest

from oracle.riskmodel import risk_model as oracle_risk_model

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("days,n,p,masked", [
    (2047, 17, 6, True), (2048, 17, 6, True), (2049, 16, 1, False), (2175, 33, 2, False), (2176, 15, 3, True),
    (2177, 1, 8, False), (2559, 40, 4, True), (2561, 40, 5, False), (2050, 129, 7, True), (2048, 4096, 2, False),
    (2048, 4097, 2, False)])
def test_long_windows(days, n, p, masked):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_22625_amd as ff
    rng = np.random.default_rng(days + n)
    Fr = rng.standard_normal((days, p)) * 0.01
    R = Fr @ rng.standard_normal((p, n)) + rng.standard_normal((days, n)) * 0.02
    M = (rng.random((days, n)) > 0.1).astype(np.uint8) if masked else None
    print(f"[case] risk days={days} n={n} p={p} masked={masked}", flush=True)
    beta, Sf, D, valid = ff.risk_model(R if M is None else np.where(M == 0, np.nan, R), Fr, mask=M)
    torch.cuda.synchronize()
    ref = oracle_risk_model(R, Fr, mask=M)
    np.testing.assert_array_equal(valid.cpu().numpy().astype(bool), ref.valid)
    np.testing.assert_allclose(beta.cpu().numpy(), ref.beta, rtol=1e-10, atol=1e-10)
    np.testing.assert_allclose(D.cpu().numpy(), ref.D, rtol=1e-10, atol=1e-20)
    np.testing.assert_allclose(Sf.cpu().numpy(), ref.Sigma_f, rtol=1e-10, atol=1e-17)
