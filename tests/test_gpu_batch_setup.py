"""Batches on either side of the number of boxes that one block plans, tiles
chosen and given, invalid boxes among them."""
import numpy as np
import pytest

import oracle
from parity import check_median, check_moments

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1211_4896_amd as tsa  # noqa: E402


@pytest.mark.parametrize("dtype", ["f32", "i16"])
@pytest.mark.parametrize("nq", [1, 63, 1023, 1024, 1025])
@pytest.mark.parametrize("tune", [None, (1024, 256, 4, 65536)])
def test_batch_setup(dtype, nq, tune):
    rng = np.random.default_rng(nq)
    host = (rng.standard_normal((24, 40, 48)) * 100).astype(np.float32 if dtype == "f32" else np.int16)
    dev = torch.from_numpy(host).to("cuda:0")
    lo = (rng.random((nq, 3)) * np.array([47, 39, 23])).astype(np.int64)
    hi = np.minimum(lo + rng.integers(1, 20, (nq, 3)), np.array([48, 40, 24]))
    boxes = np.concatenate([lo, hi], 1)
    boxes[nq // 2::97, 3] = 49  # past the cube
    want, counts = oracle.stats_boxes(host, np.minimum(boxes, [48, 40, 24, 48, 40, 24]), 16)
    print("case batch setup", dtype, nq, tune, flush=True)
    res, hists = tsa.region_batch(dev, boxes, 16, tune=tune)
    for i in range(nq):
        r = {k: res[i][k].item() for k in res.dtype.names}
        if boxes[i, 3] > 48:
            assert r["status"] == tsa.TSA_EINVAL
            continue
        what = f"{dtype} {nq} {i}"
        check_moments(r, want[i], dtype, what)
        check_median(r["median"], want[i]["median"], dtype, what)
