"""An int16 cube whose counts of values fill the halves that its sums of squares
are kept in: every value 819200 times (4096 x 4096 x 3200 voxels, 107 GB)."""
import numpy as np
import pytest

import oracle
from parity import check_hist, check_median, check_moments

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1211_4896_amd as tsa  # noqa: E402


def test_every_value_819200_times():
    times = 800
    torch.cuda.empty_cache()  # blocks that earlier cases left in torch's cache
    if torch.cuda.mem_get_info()[0] < (112 << 30):
        pytest.skip("needs 112 GiB of free device memory")
    print("case count16 large cube", flush=True)
    rng = np.random.default_rng(77)
    host = np.repeat(np.arange(-32768, 32768, dtype=np.int16), 1024)
    rng.shuffle(host)
    host = host.reshape(4, 4096, 4096)
    dev = torch.empty((4 * times, 4096, 4096), dtype=torch.int16, device="cuda:0")
    dev.view(times, 4, 4096, 4096).copy_(torch.from_numpy(host).to("cuda:0"))
    want = oracle.stats(host, 1000)
    want = {**want, "count": want["count"] * times, "nan_count": 0, "m2": want["m2"] * times}
    res, c, o = tsa.stats(dev, 1000)
    mom = tsa.moments(dev)
    del dev
    torch.cuda.empty_cache()
    check_moments(mom, want, "i16", "moments")
    check_moments(res, want, "i16", "stats")
    check_median(res["median"], want["median"], "i16", "stats")
    check_hist(c, o, want["counts"] * np.uint64(times), want["outliers"], "stats")
