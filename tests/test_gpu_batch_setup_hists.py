"""Histograms and single boxes after the one-launch set-up of a batch: every valid
box's bins on either side of the number of boxes that one block plans, and
a batch of one box, valid and not."""
import numpy as np
import pytest

import oracle
from parity import check_hist, check_median, check_moments

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1211_4896_amd as tsa  # noqa: E402


def _cube(dtype):
    rng = np.random.default_rng(4)
    return (rng.standard_normal((24, 40, 48)) * 100).astype(np.float32 if dtype == "f32" else np.int16)


def _check_all(host, boxes, tune, dtype):
    want, counts = oracle.stats_boxes(host, boxes, 16)
    res, hists = tsa.region_batch(torch.from_numpy(host).to("cuda:0"), boxes, 16, tune=tune)
    for i in range(len(boxes)):
        r = {k: res[i][k].item() for k in res.dtype.names}
        what = f"{dtype} {len(boxes)} {i} {tune}"
        check_moments(r, want[i], dtype, what)
        check_median(r["median"], want[i]["median"], dtype, what)
        check_hist(hists[i], None, counts[i], None, what)


@pytest.mark.parametrize("dtype", ["f32", "i16"])
@pytest.mark.parametrize("nq", [1, 2, 255, 256, 257, 512, 513, 1025])
@pytest.mark.parametrize("tune", [None, (1024, 256, 4, 65536)])
def test_every_histogram(dtype, nq, tune):
    print("case batch set-up histograms", dtype, nq, tune, flush=True)
    rng = np.random.default_rng(nq)
    lo = (rng.random((nq, 3)) * np.array([47, 39, 23])).astype(np.int64)
    hi = np.minimum(lo + rng.integers(1, 30, (nq, 3)), np.array([48, 40, 24]))
    _check_all(_cube(dtype), np.concatenate([lo, hi], 1), tune, dtype)


def test_one_box():
    print("case batch set-up one box", flush=True)
    host = _cube("f32")
    for box in ((0, 0, 0, 48, 40, 24), (47, 39, 23, 48, 40, 24)):
        _check_all(host, np.array([box], np.int64), None, "f32")
    res, _ = tsa.region_batch(torch.from_numpy(host).to("cuda:0"), np.array([(0, 0, 0, 49, 1, 1)], np.int64), 16)
    assert res[0]["status"] == tsa.TSA_EINVAL and res[0]["flags"] & tsa.FLAG_BAD_REGION
