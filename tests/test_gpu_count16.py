"""int16 regions answered from one count of their values, against the oracle:
both ways the counts leave a block (a table per block from 2^29 voxels on,
packed 64-bit counters below), halves that wrap, boxes, odd rows, every call."""
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


def _values(kind, n):
    rng = np.random.default_rng(31)
    if kind == "uniform":
        return rng.integers(-32768, 32768, n).astype(np.int16)
    if kind == "noise":
        return np.clip(np.rint(rng.standard_normal(n) * 300.0 + 40.0), -32768, 32767).astype(np.int16)
    if kind == "constant":
        return np.full(n, 7, np.int16)
    if kind == "constant_negative":
        return np.full(n, -5, np.int16)
    # the two halves of one counter word (7 and 7 - 32768), and the extremes
    return rng.choice(np.int16([7, 7 - 32768, 7, 7 - 32768, -32768, 32767]), n).astype(np.int16)


def _check(host, dev, region, what, times=1):
    """times: dev is host repeated that often along z (an even number of host voxels)."""
    want = oracle.stats(host, 1000, region)
    want = {**want, "count": want["count"] * times, "nan_count": 0, "m2": want["m2"] * times}
    res, c, o = tsa.stats(dev, 1000, region)
    check_moments(res, want, "i16", what)
    check_median(res["median"], want["median"], "i16", what)
    check_hist(c, o, want["counts"] * np.uint64(times), want["outliers"] * np.uint64(times), what)
    gm = tsa.median(dev, region)
    assert gm["count"] == want["count"] and gm["median"] == want["median"]
    for nb in (1, 65536):
        want = oracle.stats(host, nb, region)
        res, c, o = tsa.stats(dev, nb, region)
        check_hist(c, o, want["counts"] * np.uint64(times), want["outliers"], f"{what} {nb} bins")
    m, mad, n = oracle.mad(host, region)
    assert tsa.mad(dev, region) == (m, mad, n * times), what
    for q in (0.0, 0.5, 1.0) if times > 1 else (0.0, 0.013, 0.9, 1.0):
        v, n = oracle.quantile(host, q, region)
        assert tsa.quantile(dev, q, region) == (v, 0.0, n * times), (what, q)
        lo16 = float((int(v) + 32768) // 16 * 16 - 32768)
        assert tsa.quantile(dev, q, region, digits=1) == (lo16, 15.0, n * times), (what, q)


@pytest.mark.parametrize("kind", ["uniform", "noise", "constant", "constant_negative", "halves"])
def test_packed_counts(kind):
    _say("case count16 packed", kind)
    host = _values(kind, 1 << 24).reshape(64, 512, 512)
    _check(host, torch.from_numpy(host).to("cuda:0"), None, kind)


@pytest.mark.parametrize("shape,region", [((70, 500, 520), (3, 1, 2, 517, 499, 70)),
                                          ((66, 512, 515), (1, 0, 0, 514, 512, 66)),
                                          ((65, 511, 513), None)])
def test_boxes_and_odd_rows(shape, region):
    _say("case count16 box", shape, region)
    host = _values("noise", int(np.prod(shape))).reshape(shape)
    _check(host, torch.from_numpy(host).to("cuda:0"), region, f"{shape} {region}")


@pytest.mark.parametrize("kind,times", [("uniform", 8), ("halves", 8), ("noise", 32), ("halves", 32)])
def test_large(kind, times):
    """2^27 voxels (ranks in packed counters) and 2^29 (a table per block)."""
    _say("case count16 large", kind, times)
    host = _values(kind, 1 << 24).reshape(64, 512, 512)
    dev = torch.from_numpy(host).to("cuda:0").repeat(times, 1, 1)
    _check(host, dev, None, kind, times=times)
