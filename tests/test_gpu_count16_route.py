"""Which int16 ranks go by the count of the values: those that the passes by key
digits would read the region twice for."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1211_4896_amd as tsa  # noqa: E402


def _launches(call):
    lib = tsa.capi().lib
    lib.tsa_trace_enable.argtypes = [ctypes.c_int32, ctypes.c_int32]
    assert lib.tsa_trace_enable(1, 64) == 0
    try:
        call()
        torch.cuda.synchronize()
        buf = ctypes.create_string_buffer(1 << 16)
        assert lib.tsa_trace_read(buf, ctypes.c_size_t(len(buf))) >= 0
    finally:
        lib.tsa_trace_enable(0, 0)
    return buf.value.decode()


@pytest.mark.parametrize("digits,counted", [(1, False), (2, True), (3, True)])
def test_quantile(digits, counted):
    print("case count16 route", digits, flush=True)
    host = (np.arange(1 << 27, dtype=np.int64) * 7919 % 65536 - 32768).astype(np.int16).reshape(512, 512, 512)
    dev = torch.from_numpy(host).to("cuda:0")
    got = []
    names = _launches(lambda: got.append(tsa.quantile(dev, 0.3, digits=digits)))
    assert ("count16" in names) == counted, names
    rank = int(0.3 * (host.size - 1))  # every value 2048 times
    v = rank // 2048 - 32768
    assert got[0] == ((float(v), 0.0, host.size) if digits > 1 else (float(v & ~15), 15.0, host.size))
