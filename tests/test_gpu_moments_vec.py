"""Moments of whole float32 cubes, whose lanes take a vector's four values at once
from their first finite value on: NaN of any payload among them, lanes that find
their first finite value late or never, infinities before and after it, both
zeros, a mean far above the spread."""
import numpy as np
import pytest

import oracle
from parity import check_moments

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1211_4896_amd as tsa  # noqa: E402

STEP = 512 * 4  # voxels of a block's vectors, one a lane; a lane's next vector lies STEP on


def _cube(kind):
    rng = np.random.default_rng(3)
    x = (rng.standard_normal(9 * 4 * STEP + 5) * 3.0 + 1.0).astype(np.float32)
    u = x.view(np.uint32)
    if kind == "nan":
        m = rng.random(x.size) < 0.3
        u[m] = rng.choice(np.uint32([0x7FC00000, 0x7F800001, 0xFFFFFFFF, 0xFF800001]), int(m.sum()))
    elif kind == "late":  # a lane's first one, two or three vectors hold nothing finite
        x[:STEP] = np.nan
        x[STEP:2 * STEP:3] = np.nan
        x[STEP:2 * STEP:3] = np.inf
        x[4 * STEP:7 * STEP] = np.nan
    elif kind == "inf":
        x[5 * STEP + 77] = np.inf
    elif kind == "both":
        x[3] = -np.inf
        x[6 * STEP + 1] = np.inf
    elif kind == "zeros":
        u[:] = rng.choice(np.uint32([0, 0x80000000]), x.size)
        x[::7] = np.nan
        x[4 * STEP + 3] = 1e-42
    elif kind == "far":
        x = (rng.standard_normal(x.size) + 1e7).astype(np.float32)
        x[::11] = np.nan
    elif kind == "none":
        x[:] = np.nan
    return x


@pytest.mark.parametrize("kind", ["plain", "nan", "late", "inf", "both", "zeros", "far", "none"])
def test_vectors(kind):
    host = _cube(kind)
    print("case moments vectors", kind, flush=True)
    dev = torch.from_numpy(host).to("cuda:0")
    for n in (host.size, host.size - 5, STEP * 4, STEP * 4 + 3, 3):
        check_moments(tsa.moments(dev[:n]), oracle.moments(host[:n].reshape(1, 1, n)), "f32", f"{kind} {n}")
    check_moments(tsa.moments(dev[1:]), oracle.moments(host[1:].reshape(1, 1, -1)), "f32", f"{kind} from the second")
