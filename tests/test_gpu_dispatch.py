"""GPU: which kernel a call runs, read from its summary line on stderr, on both sides of the lines
that the host draws."""
import pytest

from synth import make_batch

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _ff():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_22625_amd as ff
    return ff


@pytest.mark.parametrize("B,line", [(100, "[ffo batch]"), (132, "[ffo lockstep]")])
def test_large_batches_take_the_lockstep_form(capfd, B, line):
    """100 rows: teams up to 4000 assets per compute unit (256 of them), lockstep beyond."""
    ff = _ff()
    batch = make_batch(B, 50, 50, seed=3, n_lo=8000, n_hi=8000)
    ff.solve_batched(batch, max_iter=64, verbose=1, raise_on_failure=False)
    assert line in capfd.readouterr().err
