"""Passes that end in one block's work on everyone's results: the block that
ends last must be the only one to run it and must see every other's, whatever
the number of blocks (around the 16 arrival groups, one block, uneven groups)."""
import sys

import numpy as np
import pytest

import oracle
from parity import check_hist, check_median, check_moments

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1211_4896_amd as tsa  # noqa: E402

CHUNK = 512 * 4 * 4  # voxels of a block's chunk (float32)


@pytest.mark.parametrize("blocks", [1, 2, 15, 16, 17, 33, 257, 800])
def test_block_counts(blocks):
    print("case launch tails", blocks, flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(blocks)
    host = (rng.standard_normal(CHUNK * blocks - 5) * 3.0 + 20.0).astype(np.float32)  # spread by the shifted moments
    host[rng.integers(0, host.size, 7)] = np.nan
    dev = torch.from_numpy(host).to("cuda:0")
    want = oracle.stats(host, 300)
    for rep in range(3):
        res, c, o = tsa.stats(dev, 300)
        check_moments(res, want, "f32", f"{blocks} {rep}")
        check_median(res["median"], want["median"], "f32", f"{blocks} {rep}")
        check_hist(c, o, want["counts"], want["outliers"], f"{blocks} {rep}")
        assert tsa.mad(dev) == oracle.mad(host)
        assert tsa.quantile(dev, 0.37)[0] == oracle.quantile(host, 0.37)[0]
