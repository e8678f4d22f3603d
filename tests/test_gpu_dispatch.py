"""GPU: which kernel a call runs, read from its summary line on stderr, on both sides of the lines
that the host draws."""
import re

import pytest

from synth import make_batch, make_multi, make_single

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _ff():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_22625_amd as ff
    return ff


def _summary(capfd, inst, **kw):
    """The fields of the summary line of one short solve."""
    ff = _ff()
    capfd.readouterr()
    ff.solve_instance(inst, max_iter=16, check_every=16, verbose=1, raise_on_failure=False, **kw)
    err = capfd.readouterr().err
    return dict(re.findall(r"(kernel|nwg|lds_k|workspace) (\S+)", err))


@pytest.mark.parametrize("n,k,m,kw,kernel", [
    (40, 2, 1, {}, "registers"),
    (900, 80, 80, {}, "registers"), (900, 80, 81, {}, "general"),             # 160 and 161 rows
    (131_072, 2, 3, {}, "registers"), (131_073, 2, 3, {}, "general"),         # 256 workgroups of 512 assets
    (65_536, 20, 29, {}, "registers"), (65_537, 80, 33, {}, "tiles"),         # ... of 256 assets; rows beyond LDS
    (32_768, 2, 3, dict(precision="fp32"), "registers"), (32_769, 2, 3, dict(precision="fp32"), "general"),
    (900, 10, 8, dict(workgroups=4), "general"), (900, 10, 8, dict(deterministic=True), "general"),
    (900, 10, 8, dict(speculative=0), "general"), (900, 10, 8, dict(noalloc=True), "registers"),
    (1400, 10, 6, dict(workgroups=1), "tiles"), (700, 10, 6, dict(workgroups=1), "general")])
def test_single_period(capfd, n, k, m, kw, kernel):
    assert _summary(capfd, make_single(n, k, m, seed=1), **kw)["kernel"] == kernel


@pytest.mark.parametrize("T,n,k,m,kw,kernel", [
    (2, 70, 3, 5, {}, "period-registers"), (32, 40, 4, 3, {}, "period-registers"), (33, 40, 4, 3, {}, "general"),
    (4, 150, 56, 56, {}, "period-registers"), (4, 150, 57, 56, {}, "general"),               # 112 and 113 rows
    (2, 16_384, 2, 3, {}, "period-registers"), (2, 16_385, 2, 3, {}, "general"),             # 256 workgroups of 64
    (4, 150, 8, 8, dict(precision="fp32"), "general"), (4, 150, 8, 8, dict(speculative=1), "general"),
    (4, 150, 8, 8, dict(deterministic=True), "general"), (4, 150, 8, 8, dict(workgroups=3), "general")])
def test_multi_period(capfd, T, n, k, m, kw, kernel):
    assert _summary(capfd, make_multi(T, n, k, m, seed=1), **kw)["kernel"] == kernel


@pytest.mark.parametrize("d,kernel", [(1.5, "registers"), (2.0, "registers"), (1.7, "general")])
def test_impact_exponents(capfd, d, kernel):
    assert _summary(capfd, make_single(300, 6, 5, seed=2, d=d))["kernel"] == kernel


def test_tiles_need_no_second_float_copy(capfd):
    """FP32 rows in tiles: the workspace holds the rows as doubles and the tiles, and less than a
    third copy (nr x n floats) besides: fifteen vectors, the breakpoint lists, an exchange slot."""
    n, k, m = 70_000, 60, 80
    f = _summary(capfd, make_single(n, k, m, seed=4), precision="fp32")
    rows, tiles = (k + m) * 8 * (n + 63), 144 * 4 * (n + 256 * 16)
    assert f["kernel"] == "tiles" and int(f["workspace"]) < rows + tiles + 25_000_000


@pytest.mark.parametrize("B,line", [(100, "[ffo batch]"), (132, "[ffo lockstep]")])
def test_large_batches_take_the_lockstep_form(capfd, B, line):
    """100 rows: teams up to 4000 assets per compute unit (256 of them), lockstep beyond."""
    ff = _ff()
    batch = make_batch(B, 50, 50, seed=3, n_lo=8000, n_hi=8000)
    ff.solve_batched(batch, max_iter=64, verbose=1, raise_on_failure=False)
    assert line in capfd.readouterr().err
