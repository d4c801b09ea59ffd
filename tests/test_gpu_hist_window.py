"""Histograms of more bins than one LDS copy holds: the window is placed from
a sample, every count is exact wherever it lies."""
import sys

import numpy as np
import pytest

import oracle
from parity import check_hist

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1211_4896_amd as tsa  # noqa: E402


@pytest.mark.parametrize("dtype", ["f32", "i16"])
@pytest.mark.parametrize("nbins", [16385, 20000, 32769, 40001, 65536])
def test_window_anywhere(dtype, nbins):
    rng = np.random.default_rng(nbins)
    shape = (23, 41, 67)
    u = rng.random(shape)
    cases = {
        "low end": u ** 6, "high end": 1.0 - u ** 6, "even": u, "both ends": np.where(u < 0.5, u / 50, 1 - u / 50),
        "outside": u + 3.0, "one value": np.full(shape, 0.37), "few": np.where(u < 0.001, u * 900, 5.0),
    }
    for what, x in cases.items():
        host = x.astype(np.float32) if dtype == "f32" else (x * 30000).clip(-32768, 32767).astype(np.int16)
        if dtype == "f32":
            host[rng.random(shape) < 0.01] = np.nan
        hi = 1.0 if dtype == "f32" else 30000.0
        dev = torch.from_numpy(host).to("cuda:0")
        for region in (None, (3, 1, 2, 66, 40, 21), (5, 5, 5, 6, 6, 6), (0, 7, 9, 67, 8, 10)):
            print("case window", dtype, nbins, what, region, flush=True)
            sys.stdout.flush()
            wc, wo = oracle.histogram(host, 0.0, hi, nbins, region)
            c, o = tsa.histogram(dev, 0.0, hi, nbins, region)
            check_hist(c, o, wc, wo, f"{dtype} {nbins} {what} {region}")
