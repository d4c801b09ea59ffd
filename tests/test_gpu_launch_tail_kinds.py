"""The work that the last block of a pass does for all of them, on data that ends
it early or crowds it, by number of blocks: no valid voxel, one value, two
values, and quantiles that stop after one or two digits."""
import math

import numpy as np
import pytest

import oracle
from parity import check_hist, check_median, check_moments

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1211_4896_amd as tsa  # noqa: E402

CHUNK = 512 * 4 * 4  # voxels of a block's chunk (float32)


def _values(kind, n):
    rng = np.random.default_rng(n)
    if kind == "none":
        return np.full(n, np.nan, np.float32)
    if kind == "one":
        return np.full(n, -2.5, np.float32)
    if kind == "two":
        return rng.choice(np.float32([-1.0, 3.0]), n).astype(np.float32)
    x = rng.standard_normal(n).astype(np.float32)
    x[rng.random(n) < 0.2] = np.nan
    return x


@pytest.mark.parametrize("kind", ["none", "one", "two", "noise"])
@pytest.mark.parametrize("blocks", [1, 16, 17, 511, 600])
def test_kinds(kind, blocks):
    print("case launch tail kinds", kind, blocks, flush=True)
    host = _values(kind, CHUNK * blocks - 3)
    dev = torch.from_numpy(host).to("cuda:0")
    want = oracle.stats(host, 77)
    for rep in range(2):
        what = f"{kind} {blocks} {rep}"
        res, c, o = tsa.stats(dev, 77)
        check_moments(res, want, "f32", what)
        check_median(res["median"], want["median"], "f32", what)
        check_hist(c, o, want["counts"], want["outliers"], what)
        assert bool(res["flags"] & tsa.FLAG_HIST_SKIPPED) == want["hist_skipped"], what
        m, mad, n = tsa.mad(dev)
        wm, wmad, wn = oracle.mad(host)
        assert n == wn and all(a == b or (math.isnan(a) and math.isnan(b)) for a, b in ((m, wm), (mad, wmad))), what
        for q in (0.0, 0.37, 1.0):
            v, n = oracle.quantile(host, q)
            for digits in (1, 2, 3):
                lo, width, count = tsa.quantile(dev, q, digits=digits)
                assert count == n, what
                if n == 0:
                    assert math.isnan(lo) and math.isnan(width), what
                else:
                    assert lo <= v <= lo + width and (digits < 3 or (lo == v and width == 0.0)), (what, q, digits)
