"""The median filter at the edges of its tiles (64 columns, 32 rows, 8 rows to a lane), in images too small for a whole
window, and with runs of NaN, infinities, equal and zero values: bit for bit against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(3, 70), (70, 3), (4, 4), (9, 5), (40, 67), (5, 66), (32, 64), (33, 65), (31, 127), (67, 130), (40, 68)])
@pytest.mark.parametrize("kind", ["plain", "few", "nan"])
def test_median_edges(H, W, kind):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1805_07920_amd as amh
    from oracle import fusion

    print("case median edges", H, W, kind, flush=True)
    rng = np.random.default_rng(H * 1000 + W)
    d = rng.uniform(2.0, 6.0, (H, W)).astype(np.float32)
    if kind == "few":  # many equal values, zeros and infinities
        d = rng.choice(np.array([0.0, 1.0, 2.0, 2.5, np.inf], np.float32), (H, W))
    if kind == "nan":
        d[rng.random((H, W)) < 0.3] = np.nan
        d[: H // 3, W // 2:] = np.nan
    with np.errstate(invalid="ignore"):
        want = fusion.median_filter4(d)
    with amh.Context() as ctx:
        got = ctx.median_filter4(torch.from_numpy(d).cuda()).cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(want))
    ok = ~np.isnan(want)
    assert np.array_equal(got[ok].view(np.uint32), want[ok].view(np.uint32))
