"""Boxes and cells that hold both zeros and nothing else: an empty range, every
value in bin 0, whichever call asks and however its work is cut."""
import numpy as np
import pytest

import oracle
from parity import check_hist, check_median, check_moments

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1211_4896_amd as tsa  # noqa: E402


def _check(r, hist, want, what):
    assert not want["hist_skipped"]
    assert not r["flags"] & tsa.FLAG_HIST_SKIPPED, what
    check_moments(r, want, "f32", what)
    check_median(r["median"], want["median"], "f32", what)
    check_hist(hist, None, want["counts"], None, what)


@pytest.mark.parametrize("nan", [False, True])
def test_both_zeros(nan):
    print("case both zeros", nan, flush=True)
    rng = np.random.default_rng(5)
    host = rng.choice(np.float32([0.0, -0.0]), (64, 64, 64)).astype(np.float32)
    if nan:
        host[rng.random(host.shape) < 0.1] = np.nan
    dev = torch.from_numpy(host).to("cuda:0")
    boxes = np.array([(0, 0, 0, 64, 64, 64), (3, 2, 1, 20, 30, 40), (8, 8, 8, 16, 16, 16)], np.int64)
    for tune in (None, (1024, 256, 4, 65536)):  # one tile a box, and many
        res, hists = tsa.region_batch(dev, boxes, 20, tune=tune)
        for i, b in enumerate(boxes):
            r = {k: res[i][k].item() for k in res.dtype.names}
            _check(r, hists[i], oracle.stats(host, 20, tuple(b)), f"box {b} {tune}")
    res, c, o = tsa.stats(dev, 20)
    _check(res, c, oracle.stats(host, 20), "stats")
    cells, hists, _ = tsa.minimap(dev, (32, 32, 16), 20)
    for i, b in enumerate(oracle.minimap_cells((64, 64, 64), (32, 32, 16))):
        r = {k: cells[i][k].item() for k in cells.dtype.names}
        _check(r, hists[i], oracle.stats(host, 20, tuple(int(v) for v in b)), f"cell {b}")
