"""int16 data in runs of one value: lanes that add eight voxels at once among
lanes that add them singly, halves that wrap under either, and the time the count
takes against that of noise."""
import ctypes
import json

import numpy as np
import pytest

import oracle
from parity import check_hist, check_median, check_moments

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1211_4896_amd as tsa  # noqa: E402


def _runs(kind, n):
    rng = np.random.default_rng(12)
    if kind == "sorted":
        return (np.arange(n, dtype=np.int64) * 65536 // n - 32768).astype(np.int16)
    # "halves": both values of one counter word, its halves wrapping in turn; "mixed": any values
    vals = np.int16([7, 7 - 32768]) if kind == "halves" else rng.integers(-32768, 32768, 1 << 16).astype(np.int16)
    lengths = rng.integers(1, 700, n // 300)
    return np.resize(np.repeat(rng.choice(vals, lengths.size), lengths), n)


@pytest.mark.parametrize("kind", ["sorted", "halves", "mixed"])
@pytest.mark.parametrize("box", [None, (1, 0, 0, 515, 511, 66)])
def test_runs(kind, box):
    print("case count16 runs", kind, box, flush=True)
    shape = (66, 511, 516)
    host = _runs(kind, int(np.prod(shape))).reshape(shape)
    dev = torch.from_numpy(host).to("cuda:0")
    want = oracle.stats(host, 1000, box)
    res, c, o = tsa.stats(dev, 1000, box)
    check_moments(res, want, "i16", kind)
    check_median(res["median"], want["median"], "i16", kind)
    check_hist(c, o, want["counts"], want["outliers"], kind)
    assert tsa.mad(dev, box) == oracle.mad(host, box)


def _count_ms(dev):
    lib = tsa.capi().lib
    lib.tsa_trace_enable.argtypes = [ctypes.c_int32, ctypes.c_int32]
    assert lib.tsa_trace_enable(1, 256) == 0
    try:
        for _ in range(8):
            tsa.median(dev)
        buf = ctypes.create_string_buffer(1 << 16)
        assert lib.tsa_trace_read(buf, ctypes.c_size_t(len(buf))) >= 0
    finally:
        lib.tsa_trace_enable(0, 0)
    return json.loads(buf.value)["count16"][2]  # the least of the launches


def test_time_of_runs():
    """One increment of a shared word for eight voxels: a sorted cube of 2^28
    voxels should take at most twice what noise takes (it took nine times with
    an increment a voxel); four times fails."""
    print("case count16 runs: time", flush=True)
    n = 1 << 28
    noise = torch.randint(-32768, 32768, (1024, 512, 512), dtype=torch.int16, device="cuda:0")
    base = _count_ms(noise)
    del noise
    runs = (torch.arange(n, device="cuda:0") // (n // 65536) - 32768).to(torch.int16).reshape(1024, 512, 512)
    assert _count_ms(runs) < 4.0 * base
