"""A small region batch on one stream while a scan of a large cube fills the chip on
another: the batch's set-up finds room beside the scan's blocks and the batch
ends long before the scan does."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1211_4896_amd as tsa  # noqa: E402


def test_batch_does_not_wait_for_the_scan():
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < (24 << 30):
        pytest.skip("needs 24 GiB of free device memory")
    print("case batch beside a scan", flush=True)
    api = tsa.capi()
    big = torch.zeros((2560, 2048, 2048), dtype=torch.int16, device="cuda:0")  # 21 GB: one pass of 3 ms and more
    big.view(-1)[::3] = 700
    small = torch.randn((64, 64, 64), device="cuda:0")
    boxes = torch.from_numpy(np.array([(2, 3, 4, 40, 41, 42)], np.int64)).to("cuda:0")
    cb, cs = tsa.cube_of(big), tsa.cube_of(small)
    wb, ws = tsa.workspace(tsa.OP_HISTOGRAM, big, None, 256), tsa.workspace(tsa.OP_REGION_BATCH, small, None, 64, 1)
    counts = torch.zeros(256, dtype=torch.int64, device="cuda:0")
    res = torch.zeros(72, dtype=torch.uint8, device="cuda:0")
    hists = torch.zeros(64, dtype=torch.int64, device="cuda:0")
    s1 = torch.cuda.Stream()
    others = [torch.cuda.Stream() for _ in range(3)]  # some stream may share the scan's hardware queue

    def scan():
        assert api.tsa_histogram(ctypes.byref(cb), None, -1000.0, 1000.0, 256, counts.data_ptr(), None, wb.data_ptr(),
                                 wb.numel(), s1.cuda_stream) == 0

    def batch(s2):
        assert api.tsa_region_batch(ctypes.byref(cs), boxes.data_ptr(), 1, 64, res.data_ptr(), hists.data_ptr(), None,
                                    ws.data_ptr(), ws.numel(), s2.cuda_stream) == 0

    def share(s2):
        begin, scanned, batched = (torch.cuda.Event(enable_timing=True) for _ in range(3))
        begin.record(s1)
        scan()
        scanned.record(s1)
        batch(s2)
        batched.record(s2)
        torch.cuda.synchronize()
        return begin.elapsed_time(batched) / begin.elapsed_time(scanned)

    for s2 in others * 2:  # code loaded, graphs captured
        share(s2)
    shares = [sorted(share(s2) for _ in range(5))[2] for s2 in others]
    assert min(shares) < 0.7, shares  # a batch that waits for the scan ends with it or after it
