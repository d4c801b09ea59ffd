"""Rows read from any element boundary, and the accumulators' whole-vector
steps, against the oracle: every width around a vector and a row's masked
ends, cubes whose rows share no alignment, values that leave the common path
(NaN of any payload, infinities, both zeros, one sign only, the value that
rounds up past the last bin)."""
import sys

import numpy as np
import pytest

import oracle
from parity import check_hist, check_median, check_moments

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1211_4896_amd as tsa  # noqa: E402


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _check(host, dev, region, dtype, what, nbins=50):
    want = oracle.stats(host, nbins, region)
    res, c, o = tsa.stats(dev, nbins, region)
    check_moments(res, want, dtype, what)
    check_median(res["median"], want["median"], dtype, what)
    if not want["hist_skipped"]:
        check_hist(c, o, want["counts"], want["outliers"], what)
    check_moments(tsa.moments(dev, region), want, dtype, what + " moments")
    assert tsa.quantile(dev, 0.7, region)[0] == oracle.quantile(host, 0.7, region)[0], what
    wc, wo = oracle.histogram(host, -1.5, 2.5, nbins, region)
    c, o = tsa.histogram(dev, -1.5, 2.5, nbins, region)
    check_hist(c, o, wc, wo, what + " histogram")


@pytest.mark.parametrize("dtype", ["f32", "i16"])
@pytest.mark.parametrize("nx", [48, 37])
def test_row_widths(dtype, nx):
    rng = np.random.default_rng(nx)
    host = (rng.standard_normal((5, 40, nx)) * (1.0 if dtype == "f32" else 900.0)).astype(
        np.float32 if dtype == "f32" else np.int16)
    if dtype == "f32":
        host[rng.random(host.shape) < 0.02] = np.nan
    dev = torch.from_numpy(host).to("cuda:0")
    boxes, keep = [], []
    for w in list(range(1, 19)) + [31, 32, 33]:
        x0 = int(rng.integers(0, nx - w + 1))
        box = (x0, 3, 1, x0 + w, 38, 5)
        _say("case row width", dtype, nx, box)
        _check(host, dev, box, dtype, f"{dtype} {nx} {box}")
        boxes.append(box)
    boxes = np.array(boxes, dtype=np.int64)
    want, counts = oracle.stats_boxes(host, boxes, 40)
    res, hists = tsa.region_batch(dev, boxes, 40)
    for i in range(len(boxes)):
        r = {k: res[i][k].item() for k in res.dtype.names}
        check_moments(r, want[i], dtype, f"batch {boxes[i]}")
        check_median(r["median"], want[i]["median"], dtype, f"batch {boxes[i]}")
        check_hist(hists[i], None, counts[i], None, f"batch {boxes[i]}")


@pytest.mark.parametrize("offset", [1, 2, 3, 5, 7])
@pytest.mark.parametrize("dtype", ["f32", "i16"])
def test_base_at_any_element(dtype, offset):
    rng = np.random.default_rng(offset)
    n = 9 * 24 * 64
    flat = (rng.standard_normal(n + offset) * (1.0 if dtype == "f32" else 900.0)).astype(
        np.float32 if dtype == "f32" else np.int16)
    host = flat[offset:].reshape(9, 24, 64)
    dev = torch.from_numpy(flat).to("cuda:0")[offset:].reshape(9, 24, 64)
    for box in (None, (0, 0, 2, 64, 24, 7), (3, 1, 0, 61, 20, 9), (4, 0, 0, 8, 24, 9)):
        _say("case base offset", dtype, offset, box)
        _check(host, dev, box, dtype, f"{dtype} offset {offset} {box}")


def _value_sets():
    rng = np.random.default_rng(8)
    n = 6000
    v = rng.standard_normal(n).astype(np.float32)
    nan_bits = v.copy()
    nan_bits.view(np.uint32)[rng.integers(0, n, 60)] = rng.choice(
        np.uint32([0x7F800001, 0x7FC00000, 0x7FFFFFFF, 0xFF800001, 0xFFC00000, 0xFFFFFFFF]), 60)
    inf = v.copy()
    inf[rng.integers(0, n, 9)] = np.inf
    return {
        "negative": -np.abs(v) - np.float32(0.5),
        "positive": np.abs(v) + np.float32(0.5),
        "zeros_negative": np.where(rng.random(n) < 0.5, np.float32(-0.0), -np.abs(v)).astype(np.float32),
        "zeros_positive": np.where(rng.random(n) < 0.5, np.float32(0.0), np.abs(v)).astype(np.float32),
        "both_zeros": rng.choice(np.float32([0.0, -0.0]), n).astype(np.float32),
        "nan_payloads": nan_bits,
        "inf": inf,
        "all_nan_but_one": np.where(np.arange(n) == 4321, np.float32(1.25), np.float32(np.nan)).astype(np.float32),
        # hi - lo times the scale rounds up to the bin count for many of these
        "past_last_bin": rng.choice(np.float32([0.1, 0.7, 3.3, 0.1 + 3.1999998]), n).astype(np.float32),
        "denormals": (rng.integers(-9, 9, n) * np.float32(1e-45)).astype(np.float32),
    }


@pytest.mark.parametrize("name", list(_value_sets().keys()))
def test_values_off_the_common_path(name):
    host = _value_sets()[name]
    dev = torch.from_numpy(host).to("cuda:0")
    for nbins in (1, 7, 300, 20000):
        _say("case values", name, nbins)
        want = oracle.stats(host, nbins)
        res, c, o = tsa.stats(dev, nbins)
        check_moments(res, want, "f32", f"{name} {nbins}")
        check_median(res["median"], want["median"], "f32", name)
        assert bool(res["flags"] & tsa.FLAG_HIST_SKIPPED) == want["hist_skipped"]
        if not want["hist_skipped"]:
            check_hist(c, o, want["counts"], want["outliers"], f"{name} {nbins}")
            for lo, hi in ((want["min"], want["max"]), (-0.75, 0.25)):
                wc, wo = oracle.histogram(host, lo, hi, nbins)
                c, o = tsa.histogram(dev, lo, hi, nbins)
                check_hist(c, o, wc, wo, f"{name} {nbins} [{lo}, {hi}]")
    cube = np.resize(host, (10, 20, 30))
    boxes = np.array([[0, 0, 0, 30, 20, 10], [1, 2, 3, 28, 19, 9]], dtype=np.int64)
    want, counts = oracle.stats_boxes(cube, boxes, 33)
    for tune in (None, (1024, 256, 4, 1 << 20, 0)):
        res, hists = tsa.region_batch(torch.from_numpy(cube).to("cuda:0"), boxes, 33, tune=tune)
        for i in range(2):
            r = {k: res[i][k].item() for k in res.dtype.names}
            check_moments(r, want[i], "f32", f"{name} batch {i}")
            check_median(r["median"], want[i]["median"], "f32", f"{name} batch {i}")
            if not r["flags"] & tsa.FLAG_HIST_SKIPPED:  # skipped for a box of both zeros: an empty range
                check_hist(hists[i], None, counts[i], None, f"{name} batch {i}")
