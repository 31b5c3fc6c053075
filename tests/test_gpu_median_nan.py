"""Median filter where windows hold NaN: every count of values from none to 16, odd and even, with ties and infinities,
against the oracle's median of the values there are."""
import numpy as np
import pytest
from test_gpu_halfpass import amh  # noqa: F401
from test_gpu_parity import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rate", [0.02, 0.3, 0.6, 0.9, 1.0])
@pytest.mark.parametrize("w,h", [(70, 41), (133, 67)])
def test_windows_with_nan(amh, rate, w, h):  # noqa: F811
    import torch
    from oracle import fusion

    say("case median nan", rate, w, h)
    rng = np.random.default_rng(int(100 * rate) + w)
    a = np.round(rng.uniform(2.0, 6.0, (h, w)) * 8).astype(np.float32) / 8  # ties
    a[rng.random((h, w)) < 0.03] = np.inf
    a[rng.random((h, w)) < rate] = np.nan
    with np.errstate(all="ignore"):
        want = fusion.median_filter4(a)
    with amh.Context() as ctx:
        got = ctx.median_filter4(torch.from_numpy(a).cuda()).cpu().numpy()
    assert np.array_equal(got, want, equal_nan=True)
