"""Performance cases: the calls a user of the library makes, at the sizes they make them.

Every case runs through the public entry points on a resident cube of the
synthetic recipe of `synth` (unit noise, compact bright sources, NULL slabs),
drawn on the GPU from the seed.  `op` says which calls one pass makes:

* query     `stats` of one small box through the Python call: an interactive
            request, where launches and host work count;
* trio      `tsa_stats` (moments + histogram over [min, max] + lower median)
            into buffers the caller keeps, of a whole cube or of a box `inset`
            voxels inside it;
* separate  `tsa_moments`, `tsa_histogram` over a fixed range, `tsa_median`;
* robust    `tsa_mad` and the 0.9-quantile: a noise estimate and a cut;
* batch     `tsa_region_batch` over `nq` boxes of log-uniform edges;
* minimap   `tsa_minimap` and the 3-sigma counts of its cells;
* spectrum  `tsa_spectrum` along sight lines.
"""
import ctypes
import math
import random

import numpy as np
import torch

import paper_1211_4896_amd as tsa

DEV = "cuda:0"
HIST_RANGE = {"f32": (-6.0, 60.0), "i16": (-32768.0, 32767.0)}
SIGMA_K, QUANTILE = 3.0, 0.9
EXACT_CHUNK = 1 << 27  # elements of a cube held in 64 bits at a time


def _cube_case(name, op, dtype, nx, ny, nz, nbins, **more):
    return {"name": name, "op": op, "dtype": dtype, "nx": nx, "ny": ny, "nz": nz, "nbins": nbins, **more}


def listed():
    return [
        # one interactive box request on a small resident cube: launch latency and host work
        _cube_case("query_box", "query", "f32", 256, 256, 256, 256, x0=101, y0=57, z0=33, lx=48, ly=40, lz=33),
        # a whole small survey cube (cache-sized)
        _cube_case("trio_256", "trio", "f32", 256, 256, 256, 1024, inset=0),
        # one GPU's share of a half-terabyte cube split 96 ways
        _cube_case("trio_1024", "trio", "f32", 1024, 1024, 1280, 4096, inset=0),
        # a large cube with the most bins a histogram takes
        _cube_case("trio_wide_bins", "trio", "f32", 2048, 2048, 1024, 65536, inset=0),
        # a large cube stored as 16-bit integers
        _cube_case("trio_int16", "trio", "i16", 2048, 2048, 2048, 4096, inset=0),
        # a box inside a survey cube whose rows are of odd length (no aligned rows)
        _cube_case("trio_odd_box", "trio", "f32", 1721, 1721, 256, 1024, inset=5),
        # the three statistics asked for one by one
        _cube_case("separate_1024", "separate", "f32", 1024, 1024, 1024, 4096),
        # noise level and a cut of a whole cube
        _cube_case("robust_1024", "robust", "f32", 1024, 1024, 1280, 0),
        # thousands of source cut-outs of every size, answered together
        _cube_case("batch_4096", "batch", "f32", 2048, 2048, 2048, 256, nq=4096, lo=8, hi=512),
        # one scheduling round of small cut-outs in the serving loop
        _cube_case("batch_64_small", "batch", "f32", 512, 512, 512, 256, nq=64, lo=8, hi=64),
        # the statistical mini-map and its local threshold
        _cube_case("minimap_30", "minimap", "f32", 1024, 1024, 1280, 64, cell=30),
        # sight lines through the cube
        _cube_case("spectrum_16384", "spectrum", "f32", 1024, 1024, 1280, 0, nrays=16384, nsamples=2560),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dims(rng, lo, hi):
    """Three edges of a cube of lo..hi voxels; half of them with rows of any length, half of a multiple of 8."""
    edge = _log_int(rng, lo, hi) ** (1.0 / 3.0)
    nx, ny, nz = (max(4, int(edge * math.exp(rng.uniform(-0.4, 0.4)))) for _ in range(3))
    return (nx if rng.random() < 0.5 else max(8, nx // 8 * 8)), ny, nz


def draw(rng):
    op = rng.choice(["query", "trio", "trio", "trio", "separate", "robust", "batch", "minimap", "spectrum"])
    c = {"op": op, "dtype": "f32" if rng.random() < 0.75 else "i16"}
    if op == "query":
        c["nx"], c["ny"], c["nz"] = _dims(rng, 1 << 21, 1 << 28)
        for a, n in (("x", c["nx"]), ("y", c["ny"]), ("z", c["nz"])):
            c["l" + a] = min(n, _log_int(rng, 8, 128))
            c[a + "0"] = rng.randrange(n - c["l" + a] + 1)
        c["nbins"] = _log_int(rng, 16, 1024)
    elif op == "trio":
        c["nx"], c["ny"], c["nz"] = _dims(rng, 1 << 15, 1 << 30)
        c["nbins"] = _log_int(rng, 16, 65536)
        c["inset"] = rng.choice([0, 0, rng.randrange(1, max(2, min(c["nx"], c["ny"], c["nz"]) // 4))])
    elif op in ("separate", "robust"):
        c["nx"], c["ny"], c["nz"] = _dims(rng, 1 << 18, 1 << 30)
        c["nbins"] = _log_int(rng, 16, 65536) if op == "separate" else 0
    elif op == "batch":
        c["nx"], c["ny"], c["nz"] = _dims(rng, 1 << 24, 1 << 31)
        c["nbins"], c["nq"] = _log_int(rng, 16, 1024), _log_int(rng, 1, 2048)
        c["lo"], c["hi"] = 8, _log_int(rng, 16, 256)
    elif op == "minimap":
        c["cell"] = _log_int(rng, 12, 64)
        c["nx"], c["ny"], c["nz"] = _dims(rng, 1 << 18, min(1 << 30, 12000 * c["cell"] ** 3))
        c["nbins"] = _log_int(rng, 16, 256)
    else:
        c["nx"], c["ny"], c["nz"] = _dims(rng, 1 << 20, 1 << 30)
        c["nbins"], c["nrays"], c["nsamples"] = 0, _log_int(rng, 1, 16384), _log_int(rng, 16, 2560)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _sources(rng, amp):
    """A 256^3 block of 200 Gaussian sources truncated at 4 sigma (their density in the recipe)."""
    blk = torch.zeros((256, 256, 256), dtype=torch.float32, device=DEV)
    for _ in range(200):
        a, s = rng.uniform(*amp), rng.uniform(2.0, 6.0)
        ctr = [rng.uniform(0, 255) for _ in range(3)]
        lo = [max(0, math.ceil(x - 4 * s)) for x in ctr]
        hi = [min(256, math.floor(x + 4 * s) + 1) for x in ctr]
        d = [torch.exp(-0.5 * ((torch.arange(l, h, device=DEV, dtype=torch.float32) - x) / s) ** 2)
             for l, h, x in zip(lo, hi, ctr)]
        blk[lo[0]:hi[0], lo[1]:hi[1], lo[2]:hi[2]] += a * d[0][:, None, None] * d[1][:, None] * d[2]
    return blk


def _cube(case, seed):
    rng = random.Random(seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    i16 = case["dtype"] == "i16"
    blk = _sources(rng, (5000.0, 50000.0) if i16 else (5.0, 50.0))
    if i16:
        blk = blk.to(torch.int32)
        cube = torch.empty((nz, ny, nx), dtype=torch.int16, device=DEV)
        for z in range(0, nz, 256):
            n = min(256, nz - z)
            slab = torch.randint(-32768, 32768, (n, ny, nx), dtype=torch.int32, device=DEV, generator=gen)
            for y in range(0, ny, 256):
                for x in range(0, nx, 256):
                    v = slab[:, y:y + 256, x:x + 256]
                    v += blk[:v.shape[0], :v.shape[1], :v.shape[2]]
            cube[z:z + n] = slab.clamp_(-32768, 32767)
        return cube
    cube = torch.empty((nz, ny, nx), dtype=torch.float32, device=DEV)
    cube.normal_(generator=gen)
    for z in range(0, nz, 256):
        for y in range(0, ny, 256):
            for x in range(0, nx, 256):
                v = cube[z:z + 256, y:y + 256, x:x + 256]
                v += blk[:v.shape[0], :v.shape[1], :v.shape[2]]
    want, have = 0.005 * cube.numel(), 0
    dims = (nz, ny, nx)
    while have < want:  # NULL slabs, 1-4 voxels thick along one axis
        ax = rng.randrange(3)
        sl, vol = [], 1
        for a, n in enumerate(dims):
            e = min(n, rng.randint(1, 4)) if a == ax else rng.randint(max(1, n // 4), n)
            o = rng.randint(0, n - e)
            sl.append(slice(o, o + e))
            vol *= e
        cube[tuple(sl)] = float("nan")
        have += vol
    return cube


def _boxes(case, seed):
    rng = np.random.default_rng(seed)
    nq = case["nq"]
    out = np.empty((nq, 6), dtype=np.int64)
    for a, n in enumerate((case["nx"], case["ny"], case["nz"])):
        e = np.clip(np.rint(np.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]), nq))).astype(np.int64), 1, n)
        o = (rng.random(nq) * (n - e + 1)).astype(np.int64)
        out[:, a], out[:, a + 3] = o, o + e
    return out


def _rays(case, seed):
    """Origins on the z = 0 face, directions within 45 degrees of +z, steps of half a voxel."""
    rng = np.random.default_rng(seed)
    n = case["nrays"]
    o = np.stack([rng.uniform(0, case["nx"] - 1, n), rng.uniform(0, case["ny"] - 1, n), np.zeros(n)], axis=1)
    th = np.arccos(rng.uniform(math.cos(math.pi / 4), 1.0, n))
    ph = rng.uniform(0, 2 * math.pi, n)
    d = 0.5 * np.stack([np.sin(th) * np.cos(ph), np.sin(th) * np.sin(ph), np.cos(th)], axis=1)
    return np.concatenate([o, d], axis=1)


def _region(case):
    """The case's box as (x0, y0, z0, x1, y1, z1), or None for the whole cube."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if case["op"] == "query":
        return (case["x0"], case["y0"], case["z0"],
                case["x0"] + case["lx"], case["y0"] + case["ly"], case["z0"] + case["lz"])
    i = case.get("inset", 0)
    return (i, i, i, nx - i, ny - i, nz - i) if i else None


def _ncells(case):
    k = case["cell"]
    return -(-case["nx"] // k) * -(-case["ny"] // k) * -(-case["nz"] // k)


def prepare(case, seed):
    """The resident cube, its descriptor, and the outputs and workspace a program keeps."""
    op, nbins = case["op"], case["nbins"]
    cube = _cube(case, seed)
    st = {"case": case, "cube": cube, "box": _region(case)}
    if op == "query":
        return st
    api = tsa.capi()
    st["c"], st["region"] = tsa.cube_of(cube), tsa.region_of(st["box"])
    st["stream"] = torch.cuda.current_stream().cuda_stream
    u8 = lambda n: torch.empty(n, dtype=torch.uint8, device=DEV)  # noqa: E731
    i64 = lambda *n: torch.empty(n, dtype=torch.int64, device=DEV)  # noqa: E731
    if op in ("trio", "separate"):
        st["out"], st["counts"], st["outl"] = torch.zeros(72, dtype=torch.uint8, device=DEV), i64(nbins), i64(2)
        if op == "trio":
            st["ws"] = tsa.workspace(tsa.OP_STATS, cube, st["box"], nbins)
        else:
            st["out2"] = torch.zeros(72, dtype=torch.uint8, device=DEV)
            ops = (tsa.OP_MOMENTS, tsa.OP_HISTOGRAM, tsa.OP_MEDIAN)
            st["ws"] = u8(max(api.tsa_workspace_bytes(o, ctypes.byref(st["c"]), None, nbins, 0) for o in ops))
    elif op == "robust":
        st["mad"] = torch.empty(3, dtype=torch.float64, device=DEV)
        st["quantile"] = torch.empty(3, dtype=torch.float64, device=DEV)
        st["ws"] = tsa.workspace(tsa.OP_MAD, cube)
    elif op == "batch":
        nq = case["nq"]
        st["boxes"] = torch.from_numpy(_boxes(case, seed)).to(DEV)
        st["out"], st["hists"] = u8(72 * nq), i64(nq, nbins)
        st["ws"] = tsa.workspace(tsa.OP_REGION_BATCH, cube, None, nbins, nq)
    elif op == "minimap":
        k, n = case["cell"], _ncells(case)
        st["out"], st["hists"], st["above"] = u8(72 * n), i64(n, nbins), i64(n)
        st["ws"] = u8(api.tsa_minimap_workspace_bytes(ctypes.byref(st["c"]), k, k, k, nbins))
    else:
        st["rays"] = torch.from_numpy(_rays(case, seed)).to(DEV)
        st["samples"] = torch.empty((case["nrays"], case["nsamples"]), dtype=torch.float64, device=DEV)
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _ok(status, what):
    if status != tsa.TSA_OK:
        raise tsa.TsaError(status, what)


def _records(buf, fields=("mean", "m2", "std", "min", "max", "median")):
    """The fields of a device buffer of result records, as views of it."""
    f, i, s = buf.view(torch.float64).view(-1, 9), buf.view(torch.int64).view(-1, 9), buf.view(torch.int32).view(-1, 18)
    at = {"mean": 2, "m2": 3, "std": 4, "min": 5, "max": 6, "median": 7}
    return {"n": i[:, 0:2], "status": s[:, 16:18] if "mean" in fields else s[:, 16], **{k: f[:, at[k]] for k in fields}}


def run(st):
    case, op, nbins = st["case"], st["case"]["op"], st["case"]["nbins"]
    if op == "query":
        res, counts, outl = tsa.stats(st["cube"], nbins, st["box"])
        return {"res": res, "counts": counts, "outliers": outl}
    api, s, c = tsa.capi(), st["stream"], ctypes.byref(st["c"])
    if op == "spectrum":
        _ok(api.tsa_spectrum(c, st["rays"].data_ptr(), case["nrays"], case["nsamples"], st["samples"].data_ptr(), s),
            "tsa_spectrum")
        return st["samples"]
    ws, ws_n = st["ws"].data_ptr(), st["ws"].numel()
    if op == "trio":
        r = ctypes.byref(st["region"]) if st["region"] is not None else None
        _ok(api.tsa_stats(c, r, nbins, st["out"].data_ptr(), st["counts"].data_ptr(), st["outl"].data_ptr(), ws, ws_n,
                          s), "tsa_stats")
        return {"res": _records(st["out"]), "counts": st["counts"], "outliers": st["outl"]}
    if op == "separate":
        lo, hi = HIST_RANGE[case["dtype"]]
        _ok(api.tsa_moments(c, None, st["out"].data_ptr(), ws, ws_n, s), "tsa_moments")
        _ok(api.tsa_histogram(c, None, lo, hi, nbins, st["counts"].data_ptr(), st["outl"].data_ptr(), ws, ws_n, s),
            "tsa_histogram")
        _ok(api.tsa_median(c, None, st["out2"].data_ptr(), ws, ws_n, s), "tsa_median")
        return {"res": _records(st["out"], ("mean", "m2", "std", "min", "max")), "counts": st["counts"],
                "outliers": st["outl"], "median": _records(st["out2"], ("median",))}
    if op == "robust":
        _ok(api.tsa_mad(c, None, st["mad"].data_ptr(), ws, ws_n, s), "tsa_mad")
        _ok(api.tsa_quantile(c, None, QUANTILE, 3, st["quantile"].data_ptr(), ws, ws_n, s), "tsa_quantile")
        return {"mad": st["mad"], "quantile": st["quantile"]}
    if op == "batch":
        _ok(api.tsa_region_batch(c, st["boxes"].data_ptr(), case["nq"], nbins, st["out"].data_ptr(),
                                 st["hists"].data_ptr(), None, ws, ws_n, s), "tsa_region_batch")
        return {"res": _records(st["out"]), "hists": st["hists"]}
    k = case["cell"]
    _ok(api.tsa_minimap(c, k, k, k, nbins, st["out"].data_ptr(), st["hists"].data_ptr(), ws, ws_n, s), "tsa_minimap")
    _ok(api.tsa_sigma_count(c, k, k, k, st["out"].data_ptr(), SIGMA_K, st["above"].data_ptr(), s), "tsa_sigma_count")
    return {"res": _records(st["out"]), "hists": st["hists"], "above": st["above"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    """Every voxel that is asked about read once, every output written once."""
    op, nbins = case["op"], case["nbins"]
    esz = 4 if case["dtype"] == "f32" else 2
    vol = case["nx"] * case["ny"] * case["nz"]
    box = _region(case) if op in ("query", "trio") else None
    if box:
        vol = (box[3] - box[0]) * (box[4] - box[1]) * (box[5] - box[2])
    if op in ("query", "trio"):
        return {"bytes": vol * esz + 72 + 8 * nbins + 16, "flops": 6 * vol}
    if op == "separate":  # three calls, each a pass of its own
        return {"bytes": 3 * vol * esz + 144 + 8 * nbins + 16, "flops": 6 * vol}
    if op == "robust":
        return {"bytes": 2 * vol * esz + 48, "flops": 4 * vol}
    if op == "batch":
        nq, lo, hi = case["nq"], case["lo"], case["hi"]
        edge = 1.0  # the mean volume of a box of log-uniform edges
        for n in (case["nx"], case["ny"], case["nz"]):
            top = min(hi, n)
            edge *= ((top - lo) + n * math.log(hi / top)) / math.log(hi / lo) if top > lo else n
        return {"bytes": nq * (edge * esz + 48 + 72 + 8 * nbins), "flops": 6 * nq * edge}
    if op == "minimap":
        n = _ncells(case)
        return {"bytes": 2 * vol * esz + n * (2 * 72 + 8 * nbins + 8), "flops": 7 * vol}
    # each ray crosses at most nz planes and reads four voxels of each
    samples = case["nrays"] * case["nsamples"]
    planes = min(case["nz"], case["nsamples"] // 2 + 1)
    return {"bytes": 8 * samples + min(vol, case["nrays"] * planes * 4) * esz + 48 * case["nrays"],
            "flops": 30 * samples}


# ---------------------------------------------------------------------------
# the same in 64 bits, with torch alone
# ---------------------------------------------------------------------------

def _chunks(cube):
    flat = cube.reshape(-1)
    for i in range(0, flat.numel(), EXACT_CHUNK):
        yield flat[i:i + EXACT_CHUNK]


def _kth(parts, k):
    """The value of 0-based rank k of the non-NaN values: bisection over the ordered codes of float32."""
    lo, hi = -(1 << 31), (1 << 31) - 1
    while lo < hi:
        mid = (lo + hi) // 2
        bits = mid if mid >= 0 else (mid ^ 0x7FFFFFFF) & 0xFFFFFFFF
        t = float(np.array([bits], dtype=np.uint32).view(np.float32)[0])
        if math.isnan(t):
            n = 0 if mid < 0 else 1 << 62
        else:
            n = sum(int((p <= t).sum()) for p in parts())
        if n > k:
            hi = mid
        else:
            lo = mid + 1
    bits = lo if lo >= 0 else (lo ^ 0x7FFFFFFF) & 0xFFFFFFFF
    return float(np.array([bits], dtype=np.uint32).view(np.float32)[0])


def _exact_values(cube, median=True):
    """(mean, m2, std, min, max, median) of the non-NaN values."""
    n, s, lo, hi = 0, 0.0, math.inf, -math.inf
    for p in _chunks(cube):
        v = p.double()
        v = v[~torch.isnan(v)]
        if v.numel():
            n, s = n + v.numel(), s + float(v.sum())
            lo, hi = min(lo, float(v.min())), max(hi, float(v.max()))
    if n == 0:
        return (math.nan,) * 6
    mean, m2 = s / n, 0.0
    for p in _chunks(cube):
        m2 += float((p.double() - mean).square().nansum())
    med = _kth(lambda: _chunks(cube), (n - 1) // 2) if median else None
    return mean, m2, math.sqrt(m2 / n), lo, hi, med


def _fields(v, scalar=False):
    keys = ("mean", "m2", "std", "min", "max", "median")
    f = (lambda x: x) if scalar else (lambda x: None if x is None else torch.tensor([x], dtype=torch.float64))
    return {"n": None, "status": None, **{k: f(x) for k, x in zip(keys, v)}}


def _exact_boxes(views):
    """Per view: mean, m2, std, min, max, median, with no host round trip per box."""
    rows = []
    inf = torch.tensor(math.inf, dtype=torch.float64, device=DEV)
    for x in views:
        x = x.reshape(-1)
        v = x.double()
        ok = ~torch.isnan(v)
        n = ok.sum()
        mean = v.nansum() / n
        m2 = (v - mean).square().nansum()
        lo, hi = torch.where(ok, v, inf).min(), torch.where(ok, v, -inf).max()
        # lower median: NaN sorts last
        med = torch.sort(x).values[((n - 1) // 2).clamp(min=0)] if x.numel() <= 1 << 20 else None
        if med is None:
            a = torch.tensor(-(1 << 31), dtype=torch.int64, device=DEV)
            b = torch.tensor((1 << 31) - 1, dtype=torch.int64, device=DEV)
            for _ in range(32):
                mid = torch.div(a + b, 2, rounding_mode="floor")
                bits = torch.where(mid >= 0, mid, mid ^ 0x7FFFFFFF)
                t = bits.to(torch.int32).view(torch.float32)
                c = torch.where(torch.isnan(t), torch.where(mid < 0, 0, 1 << 62), (x <= t).sum())
                up = c > (n - 1) // 2
                a, b = torch.where(up, a, mid + 1), torch.where(up, mid, b)
            bits = torch.where(a >= 0, a, a ^ 0x7FFFFFFF)
            med = bits.to(torch.int32).view(torch.float32)
        nan = torch.tensor(math.nan, dtype=torch.float64, device=DEV)
        row = torch.stack([mean, m2, torch.sqrt(m2 / n), lo, hi, med.double()])
        rows.append(torch.where(n > 0, row, nan))
    r = torch.stack(rows)
    return {"n": None, "status": None,
            **{k: r[:, i].contiguous() for i, k in enumerate(("mean", "m2", "std", "min", "max", "median"))}}


def _exact_minimap(cube, cell):
    nz, ny, nx = cube.shape
    cols = {k: [] for k in ("mean", "m2", "std", "min", "max", "median")}
    py, px = -(-ny // cell) * cell, -(-nx // cell) * cell
    for z in range(0, nz, cell):
        pad = torch.full((cell, py, px), math.nan, dtype=torch.float64, device=DEV)
        s = cube[z:z + cell]
        pad[:s.shape[0], :ny, :nx] = s.double()
        v = pad.view(cell, py // cell, cell, px // cell, cell).permute(1, 3, 0, 2, 4).reshape(-1, cell ** 3)
        ok = ~torch.isnan(v)
        n = ok.sum(1)
        mean = v.nansum(1) / n
        m2 = (v - mean[:, None]).square().nansum(1)
        empty = n == 0
        put = lambda k, x: cols[k].append(torch.where(empty, math.nan, x))  # noqa: E731
        put("mean", mean)
        put("m2", m2)
        put("std", torch.sqrt(m2 / n))
        put("min", torch.where(ok, v, math.inf).min(1).values)
        put("max", torch.where(ok, v, -math.inf).max(1).values)
        put("median", v.float().nanmedian(1).values.double())
    return {"n": None, "status": None, **{k: torch.cat(x) for k, x in cols.items()}}


def _exact_spectrum(cube, rays, nsamples):
    nz, ny, nx = cube.shape
    out = torch.empty((rays.shape[0], nsamples), dtype=torch.float64, device=DEV)
    i = torch.arange(nsamples, dtype=torch.float64, device=DEV)
    flat = cube.reshape(-1)
    for r0 in range(0, rays.shape[0], 1024):
        r = rays[r0:r0 + 1024]
        inside = torch.ones((r.shape[0], nsamples), dtype=torch.bool, device=DEV)
        lo, frac, up = [], [], []
        for a, n in enumerate((nx, ny, nz)):
            p = r[:, a, None] + i * r[:, 3 + a, None]
            inside &= (p >= 0) & (p <= n - 1)
            c = p.clamp(0, n - 1)
            b = c.floor().clamp(max=max(0, n - 2))
            lo.append(b.long())
            frac.append(c - b)
            up.append((b.long() + 1).clamp(max=n - 1))
        acc = torch.zeros_like(frac[0])
        for k in range(8):
            at, w = [], 1.0
            for a in range(3):
                one = (k >> a) & 1
                at.append(up[a] if one else lo[a])
                w = w * (frac[a] if one else 1.0 - frac[a])
            v = flat[(at[2] * ny + at[1]) * nx + at[0]].double()
            acc = acc + torch.where(w != 0, w * v, 0.0)
        out[r0:r0 + 1024] = torch.where(inside, acc, math.nan)
    return out


def exact(case, seed):
    op = case["op"]
    cube = _cube(case, seed)
    box = _region(case)
    if box:
        cube = cube[box[2]:box[5], box[1]:box[4], box[0]:box[3]].contiguous()
    if op == "query":
        v = _fields(_exact_values(cube), scalar=True)
        del v["n"]
        return {"counts": None, "outliers": None, "res": {"count": None, "nan_count": None, "flags": None, **v}}
    if op == "trio":
        return {"res": _fields(_exact_values(cube)), "counts": None, "outliers": None}
    if op == "separate":
        v = _fields(_exact_values(cube))
        med = v.pop("median")
        return {"res": v, "counts": None, "outliers": None, "median": {"n": None, "status": None, "median": med}}
    if op == "robust":
        n = sum(int((~torch.isnan(p)).sum()) if p.is_floating_point() else p.numel() for p in _chunks(cube))
        m = _kth(lambda: _chunks(cube), (n - 1) // 2)
        q = _kth(lambda: _chunks(cube), int(math.floor(QUANTILE * (n - 1))))
        f = lambda p: (p.float() - m).abs_()  # noqa: E731
        mad = _kth(lambda: (f(p) for p in _chunks(cube)), (n - 1) // 2)
        t = lambda *v: torch.tensor(v, dtype=torch.float64)  # noqa: E731
        return {"mad": t(m, mad, n), "quantile": t(q, 0.0, n)}
    if op == "batch":
        b = _boxes(case, seed)
        return {"res": _exact_boxes(cube[z0:z1, y0:y1, x0:x1] for x0, y0, z0, x1, y1, z1 in b.tolist()), "hists": None}
    if op == "minimap":
        return {"res": _exact_minimap(cube, case["cell"]), "hists": None, "above": None}
    return _exact_spectrum(cube, torch.from_numpy(_rays(case, seed)).to(DEV), case["nsamples"])
