"""Bracketed ranks where the sample grows with the region (2^20 voxels from 7.0e9 on,
2^22 from 1.4e10) and the digits behind them above 2.68e10: a slab of odd count
repeated along z, whose ranks are the slab's own."""
import ctypes
import json

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1211_4896_amd as tsa  # noqa: E402

SHAPE = (16, 2048, 2048)  # 2^26 voxels


def _slab():
    rng = np.random.default_rng(23)
    x = (rng.standard_normal(SHAPE, dtype=np.float32) * np.float32(0.1) + np.float32(100.0)).reshape(-1)
    x[rng.integers(0, x.size, 500000)] = np.nan
    if np.count_nonzero(x == x) % 2 == 0:
        x[np.flatnonzero(x == x)[0]] = np.nan
    return x.reshape(SHAPE)


def _traced(call):
    lib = tsa.capi().lib
    lib.tsa_trace_enable.argtypes = [ctypes.c_int32, ctypes.c_int32]
    assert lib.tsa_trace_enable(1, 256) == 0
    try:
        out = call()
        buf = ctypes.create_string_buffer(1 << 16)
        assert lib.tsa_trace_read(buf, ctypes.c_size_t(len(buf))) >= 0
    finally:
        lib.tsa_trace_enable(0, 0)
    return out, json.loads(buf.value)


@pytest.mark.parametrize("times,bracketed", [(112, True), (300, True), (400, False)])
def test_repeated_slab(times, bracketed):
    torch.cuda.empty_cache()  # blocks that earlier cases left in torch's cache
    nbytes = 4 * times * int(np.prod(SHAPE))
    if torch.cuda.mem_get_info()[0] < nbytes + (4 << 30):
        pytest.skip(f"needs {nbytes >> 30} GiB of free device memory")
    print("case bracket large", times, flush=True)
    host = _slab()
    v = np.sort(host[host == host])
    n = v.size
    dev = torch.empty((times, *SHAPE), dtype=torch.float32, device="cuda:0")
    dev.copy_(torch.from_numpy(host).to("cuda:0"))
    dev = dev.view(times * SHAPE[0], SHAPE[1], SHAPE[2])
    med, launches = _traced(lambda: tsa.median(dev))
    assert ("bracket" in launches) == bracketed
    if bracketed:
        assert launches["level1"][1] < 0.2  # the bracket answered: the digits end at once
    assert med["count"] == n * times and med["nan_count"] == (host.size - n) * times
    assert med["median"] == float(v[(n - 1) // 2])
    for q in (0.001, 0.9):
        k = oracle.quantile_rank(q, n * times)
        assert tsa.quantile(dev, q) == (float(v[k // times]), 0.0, n * times), q
    dev_sorted = np.sort(np.abs(v - v[(n - 1) // 2]))
    assert tsa.mad(dev) == (float(v[(n - 1) // 2]), float(dev_sorted[(n - 1) // 2]), n * times)
    del dev
    torch.cuda.empty_cache()
