"""Ranks of large float32 regions from a bracket: values that many voxels
share, both zeros, infinities, NaN, ranks at either end, samples that mislead
(the rank outside the bounds, more voxels between them than the list holds)."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1211_4896_amd as tsa  # noqa: E402

SIDE, TIMES = 256, 16  # host 256^2 x 128, repeated along z: 2^27 voxels
QS = (0.0, 1e-7, 0.013, 0.5, 0.9, 0.999999, 1.0)


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _host(kind):
    rng = np.random.default_rng(5)
    n = SIDE * SIDE * 128
    x = rng.standard_normal(n).astype(np.float32)
    u = rng.random(n)
    if kind == "noise":
        x[u < 0.01] = np.nan
    elif kind == "zeros":  # the median among the zeros of either sign
        x = np.where(u < 0.3, -np.abs(x), np.where(u < 0.48, np.float32(-0.0), np.where(u < 0.7, np.float32(0.0), np.abs(x))))
    elif kind == "plus_zero":
        x = np.where(u < 0.3, -np.abs(x), np.where(u < 0.36, np.float32(-0.0), np.where(u < 0.7, np.float32(0.0), np.abs(x))))
    elif kind == "ten":
        x = np.floor(u * 10)
    elif kind == "hundred":
        x = np.floor(u * 100) - 50
    elif kind == "constant":
        x[:] = 3.25
    elif kind == "infinities":
        x = np.where(u < 0.45, -np.inf, np.where(u < 0.5, x, np.inf))
    elif kind == "minus_infinity":
        x = np.where(u < 0.6, -np.inf, x)
    elif kind == "nan":
        x[:] = np.nan
    elif kind == "few":
        x[u > 1e-4] = np.nan
    elif kind == "denormal":
        x = (rng.integers(-2000, 2000, n) * np.float64(1.4e-45)).astype(np.float32)
    elif kind == "coarse":  # few keys a standard deviation, none a large share
        x = x * np.float32(0.1) + np.float32(1000.0)
    elif kind == "ramp":
        x = np.arange(n, dtype=np.float32) * np.float32(-0.5)
    return np.ascontiguousarray(x.astype(np.float32).reshape(128, SIDE, SIDE))


def _same(got, want, what):
    got, want = np.float32(got), np.float32(want)
    assert got.tobytes() == want.tobytes() or (np.isnan(got) and np.isnan(want)), (what, got, want)


@pytest.mark.parametrize("kind", ["noise", "zeros", "plus_zero", "ten", "hundred", "constant", "infinities",
                                  "minus_infinity", "nan", "few", "denormal", "coarse", "ramp"])
def test_repeated_values(kind):
    host = _host(kind)
    dev = torch.from_numpy(host).to("cuda:0").repeat(TIMES, 1, 1)
    valid = host[~np.isnan(host)]
    u = valid.view(np.uint32)
    order = np.sort(np.where(u >> 31, ~u, u | np.uint32(0x80000000)))
    back = np.where(order >> 31, order & np.uint32(0x7FFFFFFF), ~order).astype(np.uint32).view(np.float32)
    n = valid.size * TIMES
    _say("case median", kind)
    r = tsa.median(dev)
    assert r["count"] == n and r["nan_count"] == dev.numel() - n
    _same(r["median"], back[((n - 1) // 2) // TIMES] if n else np.nan, kind)
    for q in QS:
        _say("case quantile", kind, q)
        v, w, c = tsa.quantile(dev, q)
        assert c == n
        if n:
            assert w == 0.0
            _same(v, back[oracle.quantile_rank(q, n) // TIMES], (kind, q))
        else:
            assert np.isnan(v)
    _say("case mad", kind)
    m, d, c = oracle.mad(host)
    gm, gd, gc = tsa.mad(dev)
    assert gc == n
    _same(gm, m, kind)
    _same(gd, d, kind)


def _sampled(volume, ns=1 << 18):
    s = np.arange(ns, dtype=np.uint64)
    run = np.uint64(volume // ns)
    return (s * run + ((run * ((s * np.uint64(0x9E3779B1)) & np.uint64(0xFFFFFFFF))) >> np.uint64(32))).astype(np.int64)


@pytest.mark.parametrize("kind", ["outside_above", "outside_below", "overflow"])
def test_sample_misleads(kind):
    dev = torch.randn(TIMES * 128, SIDE, SIDE, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(3))
    at = torch.from_numpy(_sampled(dev.numel())).to("cuda:0")
    if kind == "overflow":
        dev *= 1e-3
        dev.view(-1)[at] = torch.linspace(-50, 50, at.numel(), device="cuda:0")
    else:
        dev.view(-1)[at] = 1e6 if kind == "outside_above" else -1e6
    flat = dev.view(-1).sort().values
    n = flat.numel()
    for q in (0.3, 0.5, 0.7):
        _say("case misled", kind, q)
        assert tsa.quantile(dev, q) == (flat[oracle.quantile_rank(q, n)].item(), 0.0, n)
    m = flat[(n - 1) // 2]
    assert tsa.median(dev)["median"] == m.item()
    d = (dev.view(-1) - m).abs().sort().values[(n - 1) // 2]
    assert tsa.mad(dev) == (m.item(), d.item(), n)


@pytest.mark.parametrize("box", [None, (1, 0, 0, 513, 515, 517), (1, 2, 1, 513, 515, 517)])
def test_boxes_of_odd_rows(box):
    dev = torch.randn(517, 515, 513, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(4))
    b = box or (0, 0, 0, 513, 515, 517)
    part = dev[b[2]:b[5], b[1]:b[4], b[0]:b[3]].reshape(-1)
    flat = part.sort().values
    n = flat.numel()
    _say("case box", box)
    m = flat[(n - 1) // 2]
    assert tsa.median(dev, box)["median"] == m.item()
    assert tsa.quantile(dev, 0.9, box) == (flat[oracle.quantile_rank(0.9, n)].item(), 0.0, n)
    d = (part - m).abs().sort().values[(n - 1) // 2]
    assert tsa.mad(dev, box) == (m.item(), d.item(), n)
