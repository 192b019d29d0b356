"""Timed cases of the search and of its candidate classifier.

Each case is one pass through the library's public entry points as a program
that uses them makes it: a search plan (or batch, stream, multi-timescale plan,
classifier) is created once, inputs are on the GPU, and a pass runs the call
and takes its results.

listed() holds the fixed cases, draw(rng) makes one more over the same ranges,
prepare(case, seed) builds what a program holds before the call, run(state) is
the pass, work(case) counts the bytes and operations that the method cannot do
without, and exact(case, seed) gives the computed outputs in 64 bits.
"""
import math

import numpy as np
import torch

from paper_2510_18136_amd import nsfrb, synth

DT_MS, K_DM_MS = 134.2, 4.15
TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
NBYTES = {"f32": 4, "f16": 2, "bf16": 2}
WIDTHS_16 = "1,2,4,8,16"
WIDTHS_1200 = "1,2,4,8,16,32,64,128,256,512,1024,1200"


# ------------------------------------------------------------------ the cases
def _search(name, nx, ny, n_sub, n_time, n_dm, dm_max, widths, raw="f32", store="f32", k=10):
    return {"name": name, "kind": "search", "nx": nx, "ny": ny, "n_sub": n_sub, "n_time": n_time, "n_dm": n_dm,
            "dm_max": dm_max, "widths": widths, "raw": raw, "store": store, "k": k}


def listed():
    return [
        # the smallest search (32 x 32 pixels, 64 samples): one call answered at once, latency and launches
        _search("search_tiny", 32, 32, 4, 64, 8, 1000.0, WIDTHS_16),
        # a small search with no round size: odd sub-bands and samples, BF16 store, a width that is no power of two
        _search("search_odd", 75, 61, 13, 333, 24, 2000.0, "1,2,4,8,16,32,64,100", store="bf16", k=100),
        # an ordinary image cube of a length that is no multiple of 64 samples
        _search("search_ragged", 201, 150, 16, 1500, 16, 4000.0, "1,2,4,8,16,32,64,128,300"),
        # the paper's own grid (16 DM trials, widths 1-16) on a 16-bit cube, stored in 16 bits
        _search("search_paper_f16", 256, 256, 16, 2048, 16, 4000.0, WIDTHS_16, raw="f16", store="f16"),
        # the survey search: 32 DM trials, widths 1-1200, FP32 throughout; the largest call
        _search("search_survey", 256, 256, 16, 2048, 32, 4000.0, WIDTHS_1200),
        # the training driver's cubes: 16 equal raw cubes normalised and searched in one batch
        {"name": "batch_training", "kind": "batch", "n_cubes": 16, "shapes": 0, "side_lo": 64, "side_hi": 64,
         "t_lo": 256, "t_hi": 256, "layout": "tsp"},
        # the process server's batch: cubes of uneven size, already normalised, FP16
        {"name": "batch_uneven", "kind": "batch", "n_cubes": 10, "shapes": 5, "side_lo": 64, "side_hi": 256,
         "t_lo": 256, "t_hi": 4096, "layout": "pst"},
        # real time: 25 new samples enter the ring and the 2048-sample window is searched
        {"name": "stream_push", "kind": "stream", "nx": 128, "ny": 128, "n_sub": 16, "n_time": 2048, "n_dm": 32,
         "dm_max": 4000.0, "widths": WIDTHS_1200, "store": "f32", "chunk": 25},
        # the paper's three sampling timescales (1, 5 and 75 samples) of one cube
        {"name": "multiscale", "kind": "multiscale", "nx": 128, "ny": 128, "n_sub": 16, "n_time": 2048, "n_dm": 32,
         "dm_max": 4000.0, "widths": WIDTHS_16, "store": "f32"},
        # candidates' cutouts for one classifier batch, out of FP16 cubes
        {"name": "cutouts", "kind": "cutouts", "n": 64, "n_cubes": 16, "side": 64, "n_time": 256, "store": "f16"},
        # the classifier on one batch of candidates
        {"name": "infer", "kind": "infer", "n": 64, "t": 64, "ny": 32},
        # one training step (forward, backward, Adam) on one batch
        {"name": "train", "kind": "train", "n": 64, "t": 64, "ny": 32},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _fit_sub(n_time, store, n_sub):
    """Sub-bands whose rows of n_time samples (with the longest delay) fit one workgroup's LDS."""
    return max(2, min(n_sub, 150000 // ((n_time + 230) * NBYTES[store])))


def _draw_widths(rng, n_time):
    if n_time > 2400 or rng.random() < 0.4:
        return WIDTHS_16
    top = max(4, n_time // 2)
    w = [1 << i for i in range(top.bit_length()) if (1 << i) <= top]
    return ",".join(map(str, w + [rng.randint(3, top) | 1]))


def draw(rng):
    kind = rng.choice(["search"] * 5 + ["batch"] * 2 + ["stream", "multiscale", "cutouts", "infer", "train"])
    if kind in ("search", "stream", "multiscale"):
        n_time = _log(rng, 48, 4096) if kind == "search" else _log(rng, 200, 2048)
        store = rng.choice(["f32", "f32", "f16", "bf16"])
        n_sub = _fit_sub(n_time, store, rng.choice([4, 8, 16, 16, rng.randint(3, 16)]))
        pix = _log(rng, 1000, min(65536, 200000000 // (n_sub * n_time)))
        nx = max(8, int(round(math.sqrt(pix) * rng.uniform(0.8, 1.25))))
        case = {"kind": kind, "nx": nx, "ny": max(8, pix // nx), "n_sub": n_sub, "n_time": n_time,
                "n_dm": rng.choice([8, 16, 32, rng.randint(5, 32)]), "dm_max": float(rng.choice([1000, 2000, 4000])),
                "widths": _draw_widths(rng, n_time), "store": store}
        if kind == "search":
            case["raw"] = rng.choice(["f32", "f32", "f16", "bf16"])
            case["k"] = rng.choice([10, 100])
        elif kind == "stream":
            case["chunk"] = rng.choice([25, 25, rng.randint(10, 50)])
        else:
            case["widths"] = WIDTHS_16
        return case
    if kind == "batch":
        lo = _log(rng, 32, 96)
        t_lo = _log(rng, 128, 512)
        return {"kind": kind, "n_cubes": rng.randint(3, 12), "shapes": rng.randint(1, 1 << 20), "side_lo": lo,
                "side_hi": lo + rng.randint(0, 100), "t_lo": t_lo, "t_hi": t_lo * rng.randint(1, 8),
                "layout": rng.choice(["tsp", "pst"])}
    if kind == "cutouts":
        return {"kind": kind, "n": rng.randint(3, 64), "n_cubes": rng.randint(1, 16), "side": _log(rng, 40, 128),
                "n_time": _log(rng, 100, 600), "store": rng.choice(["f32", "f16", "bf16"])}
    return {"kind": kind, "n": _log(rng, 2, 48), "t": rng.choice([64, 64, rng.randint(16, 64)]),
            "ny": rng.choice([32, 32, rng.randint(9, 32)])}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _widths(case):
    return [int(w) for w in case["widths"].split(",")]


def _freqs(n_sub):
    return np.linspace(1.311, 1.499, n_sub)


def _dms(case):
    return np.linspace(0.0, case["dm_max"], case["n_dm"])


def _sky(case, n_time, seed, dtype, amp=1.0):
    """A raw cube [n_time][n_sub][pixels]: noise of a sigma per pixel, dispersed pulses, zero-DM spikes and a stripe."""
    ns, npix = case["n_sub"], case["nx"] * case["ny"]
    x = torch.empty((n_time, ns, npix), dtype=dtype, device="cuda")
    g, rng = _gen(seed), np.random.default_rng(seed)
    sig = torch.from_numpy(rng.uniform(0.8, 1.2, npix).astype(np.float32)).cuda()
    for t in range(0, n_time, 64):
        n = min(64, n_time - t)
        x[t:t + n] = (torch.randn((n, ns, npix), generator=g, device="cuda") * sig).to(dtype)
    freqs = _freqs(ns)
    for p in rng.choice(npix, size=min(40, npix), replace=False):
        w = int(round(math.exp(rng.uniform(0.0, math.log(max(2, n_time // 2))))))
        off = synth.arrival_offsets(rng.uniform(0.0, case["dm_max"]), freqs, freqs.max(), DT_MS)
        t0 = int(rng.integers(0, max(1, n_time - w)))
        a = amp * rng.uniform(6.0, 50.0) / math.sqrt(w * ns)
        for s in range(ns):
            x[t0 + int(off[s]):t0 + int(off[s]) + w, s, int(p)] += a
    for t in rng.choice(n_time, size=min(20, max(1, n_time // 100)), replace=False):
        x[int(t)] += (5.0 * sig).to(dtype)
    x[:, int(rng.integers(0, ns))] += (5.0 * sig).to(dtype)
    return x


def _config(case, raw, store, n_time=None, layout="tsp", norm="pixel_subband", k=10):
    return nsfrb.SearchConfig(case["nx"], case["ny"], n_time or case["n_time"], _freqs(case["n_sub"]), _dms(case),
                              _widths(case), in_dtype=raw, store_dtype=store, norm=norm, layout=layout,
                              snr_threshold=6.0, max_candidates=k)


def _batch_shapes(case):
    """(side, sub-bands, samples) of the cubes; shapes 0: all alike, 16 sub-bands."""
    rng = np.random.default_rng(case["shapes"])
    out = []
    for _ in range(case["n_cubes"]):
        side, t = (int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))
                   for lo, hi in ((case["side_lo"], case["side_hi"]), (case["t_lo"], case["t_hi"])))
        out.append((side, 16 if case["shapes"] == 0 else int(rng.choice([8, 16])), t))
    return out


def _batch_cases(case):
    return [{"nx": side, "ny": side, "n_sub": ns, "n_time": t, "n_dm": 8, "dm_max": 1000.0, "widths": WIDTHS_16}
            for side, ns, t in _batch_shapes(case)]


def _batch_cube(case, c, i, seed):
    x = _sky(c, c["n_time"], seed * 1000 + i, torch.float32)
    if case["layout"] == "pst":
        x = x.permute(2, 1, 0).contiguous().to(torch.float16)
    return x


class _Buffer:
    """A device buffer of the library's, as torch sees it; keeps its owner alive."""

    def __init__(self, ptr, shape, typestr, owner):
        self.owner = owner
        self.__cuda_array_interface__ = {"data": (int(ptr), False), "shape": tuple(shape), "typestr": typestr,
                                         "version": 2}


def _maps(search, owner):
    """The S/N and TOA maps [n_dm][n_width][pixels] that a search leaves on the GPU."""
    import ctypes
    s, t = ctypes.c_void_p(), ctypes.c_void_p()
    nsfrb.check(nsfrb.lib().nsfrb_maps_device(search.h, ctypes.byref(s), ctypes.byref(t)))
    shape = (search.cfg.dms.size, search.cfg.widths.size, search.cfg.n_pix)
    return (torch.as_tensor(_Buffer(s.value, shape, "<f4", owner), device="cuda"),
            torch.as_tensor(_Buffer(t.value, shape, "<i4", owner), device="cuda"))


def _candidates(recs, total):
    keys = ("x", "y", "dm_index", "width_index", "toa") + (("scale",) if recs and "scale" in recs[0] else ())
    return {"index": np.array([[r[k] for k in keys] for r in recs], np.int64).reshape(len(recs), -1),
            "snr": np.array([r["snr"] for r in recs], np.float32), "total": int(total)}


def _stream_chunks(case, seed):
    """Samples that arrive in batches of `chunk`: enough to fill the ring, then three more batches."""
    n_fill = -(-case["n_time"] // case["chunk"])
    return n_fill, _sky(case, (n_fill + 3) * case["chunk"], seed, torch.float32)


def _cutout_plan(case, seed):
    rng = np.random.default_rng(seed)
    c = {"nx": case["side"], "ny": case["side"], "n_sub": 16, "n_time": case["n_time"], "n_dm": 8, "dm_max": 1000.0,
         "widths": WIDTHS_16}
    desc = [(int(rng.integers(0, case["n_cubes"])), int(rng.integers(0, case["side"])),
             int(rng.integers(0, case["side"])), int(rng.integers(0, 8)), int(rng.integers(0, case["n_time"] - 8)))
            for _ in range(case["n"])]
    return c, desc


def _cutout_cubes(case, seed):
    g = _gen(seed)
    shape = (case["side"] * case["side"], 16, case["n_time"])
    return [torch.randn(shape, generator=g, device="cuda").to(TORCH[case["store"]]) for _ in range(case["n_cubes"])]


def _cutout_batch(case, seed):
    """Cutouts [n][t][y][32][16] in BF16 (unit noise, a pulse at the centre of half of them) and labels."""
    g, rng = _gen(seed), np.random.default_rng(seed)
    n, t, ny = case["n"], case["t"], case["ny"]
    x = torch.randn((n, t, ny, 32, 16), generator=g, device="cuda")
    y = np.ones(n, np.float32)
    for i in range(0, n, 2):
        w = int(rng.integers(1, max(2, t // 4)))
        x[i, t // 2:t // 2 + w, ny // 2, 16] += rng.uniform(5.0, 50.0) / math.sqrt(16 * w)
        y[i] = 0.0
    return x.to(torch.bfloat16), torch.from_numpy(y).cuda()


CONV_IN = (16, 32, 32, 32)


def _parameters(seed):
    """A weight vector in the library's layout: He-uniform convolutions, uniform head, small biases."""
    rng, out = np.random.default_rng(seed + 77), []
    for cin in CONV_IN:
        lim = math.sqrt(6.0 / (27 * cin))
        out += [rng.uniform(-lim, lim, 32 * 27 * cin), rng.uniform(-0.02, 0.02, 32)]
    out += [rng.uniform(-0.3, 0.3, 32 * 64), rng.uniform(-0.02, 0.02, 32), rng.uniform(-0.4, 0.4, 32), np.zeros(1)]
    return np.concatenate(out).astype(np.float32)


# ------------------------------------------------------------------ prepare and run
def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind}
    if kind == "search":
        st["x"] = _sky(case, case["n_time"], seed, TORCH[case["raw"]])
        st["search"] = nsfrb.Search(_config(case, case["raw"], case["store"], k=case["k"]))
        st["maps"] = _maps(st["search"], st["search"])
    elif kind == "batch":
        cs = _batch_cases(case)
        st["x"] = [_batch_cube(case, c, i, seed) for i, c in enumerate(cs)]
        pst = case["layout"] == "pst"
        st["batch"] = nsfrb.Batch([_config(c, "f16" if pst else "f32", "f16", layout=case["layout"],
                                           norm="none" if pst else "pixel_subband") for c in cs])
        st["ptrs"] = [x.data_ptr() for x in st["x"]]
    elif kind == "stream":
        n_fill, x = _stream_chunks(case, seed)
        st["x"], st["chunk"] = x, case["chunk"]
        st["stream"] = nsfrb.Stream(_config(case, "f32", case["store"]), chunk=case["chunk"])
        for k in range(n_fill):
            st["stream"].push(x[k * case["chunk"]:].data_ptr())
        st["next"], st["first"], st["end"] = n_fill, n_fill, n_fill + 3
        st["maps"] = _maps(st["stream"].search(), st["stream"])
    elif kind == "multiscale":
        st["x"] = _sky(case, case["n_time"], seed, torch.float32)
        st["ms"] = nsfrb.MultiScale(_config(case, "f32", case["store"]))
        st["maps"] = [_maps(st["ms"].scale(k), st["ms"]) for k in range(3)]
    elif kind == "cutouts":
        c, st["desc"] = _cutout_plan(case, seed)
        st["case"] = dict(case)
        st["z"] = _cutout_cubes(case, seed)
        st["clf"] = nsfrb.Classifier(max_batch=case["n"])
        st["delays"] = _config(c, case["store"], case["store"]).delays()
        st["out"] = torch.empty((case["n"], 64, 32, 32, 16), dtype=torch.bfloat16, device="cuda")
        st["ptrs"] = [z.data_ptr() for z in st["z"]]
    else:
        st["n"] = case["n"]
        st["x"], st["y"] = _cutout_batch(case, seed)
        st["clf"] = nsfrb.Classifier(max_batch=case["n"], n_time=case["t"], ny=case["ny"])
        st["clf"].set_params(_parameters(seed))
        st["prob"] = torch.empty(case["n"], dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    return st


def run(st):
    kind = st["kind"]
    if kind == "search":
        st["search"].run(st["x"].data_ptr())
        recs, total, _ = st["search"].candidates()
        return {"snr": st["maps"][0], "toa": st["maps"][1], "candidates": _candidates(recs, total)}
    if kind == "batch":
        st["batch"].run(st["ptrs"])
        out = []
        for i in range(len(st["ptrs"])):
            s, d, w, t = st["batch"].best(i)
            out.append({"snr": s, "trial": np.stack([d, w, t])})
        return out
    if kind == "stream":
        k = st["next"]
        st["next"] = k + 1 if k + 1 < st["end"] else st["first"]
        r = st["stream"].push(st["x"][k * st["chunk"]:].data_ptr())
        return {"snr": st["maps"][0], "toa": st["maps"][1],
                "candidates": _candidates([r["cand"]] if r["has_candidate"] else [], r["has_candidate"])}
    if kind == "multiscale":
        st["ms"].run(st["x"].data_ptr())
        recs, total, _ = st["ms"].candidates()
        return {"snr": [m[0] for m in st["maps"]], "toa": [m[1] for m in st["maps"]],
                "candidates": _candidates(recs, total)}
    if kind == "cutouts":
        c = st["case"]
        st["clf"].cutouts(st["ptrs"], c["store"], c["side"], c["side"], 16, c["n_time"], st["delays"], st["desc"],
                          st["out"].data_ptr())
        return st["out"]
    if kind == "infer":
        st["clf"].infer(st["x"].data_ptr(), st["n"], st["prob"].data_ptr())
        return st["prob"]
    loss = st["clf"].train_step(st["x"].data_ptr(), st["y"].data_ptr(), st["n"])
    return {"loss": float(loss), "grads": st["clf"].grads()}


# ------------------------------------------------------------------ work
def _search_work(case, n_time, n_dm, dt_ms, dm_max, raw, store, tsp=True):
    """Bytes and operations of one search: the raw cube is read, the normalised cube written and read back, the maps
    written; per (pixel, DM) the de-dispersion adds and, per width, one add and one compare per window."""
    ns, npix, widths = case["n_sub"], case["nx"] * case["ny"], _widths(case)
    cells = float(npix) * ns * n_time
    f = _freqs(ns)
    ops = 0.0
    for dm in np.linspace(0.0, dm_max, n_dm):
        length = n_time - int(synth.arrival_offsets(dm, f, f.max(), dt_ms).max())
        if length > 0:
            ops += (ns - 1) * length + sum(2 * max(0, length - w + 1) for w in widths)
    by = cells * (NBYTES[raw] + 2 * NBYTES[store] if tsp else NBYTES[store]) + 8.0 * n_dm * len(widths) * npix
    return {"bytes": by, "flops": ops * npix + (8.0 * cells if tsp else 0.0)}


def work(case):
    kind = case["kind"]
    if kind in ("search", "stream"):
        w = _search_work(case, case["n_time"], case["n_dm"], DT_MS, case["dm_max"], case.get("raw", "f32"),
                         case["store"])
        if kind == "stream":
            w["bytes"] += 8.0 * case["chunk"] * case["n_sub"] * case["nx"] * case["ny"]
        return w
    if kind == "batch":
        ws = [_search_work(c, c["n_time"], 8, DT_MS, 1000.0, "f32", "f16", case["layout"] == "tsp")
              for c in _batch_cases(case)]
        return {k: sum(w[k] for w in ws) for k in ("bytes", "flops")}
    if kind == "multiscale":
        total = {"bytes": 0.0, "flops": 0.0}
        cells = 4.0 * case["nx"] * case["ny"] * case["n_sub"]
        for f, scale in ((1, 1.0), (5, 5.0), (75, 0.0)):
            n_dm = case["n_dm"] if scale else 1
            w = _search_work(case, case["n_time"] // f, n_dm, DT_MS * f, case["dm_max"] * scale, "f32", case["store"])
            if f > 1:                                 # the binned cube, written once (the raw cube is read once)
                w["bytes"] += cells * (case["n_time"] // f)
            total = {k: total[k] + w[k] for k in total}
        return total
    if kind == "cutouts":
        cells = case["n"] * 64.0 * 32 * 32 * 16
        return {"bytes": cells * (2 + NBYTES[case["store"]]), "flops": cells}
    pos = float(case["n"] * case["t"] * case["ny"] * 32)
    conv = [2.0 * 27 * 32 * cin * pos for cin in CONV_IN]
    if kind == "infer":
        return {"bytes": pos * 2 * (16 + 32 * 8), "flops": sum(conv)}
    return {"bytes": pos * 2 * (16 * 2 + 32 * 4 * 5), "flops": 2 * sum(conv) + sum(conv[1:])}


# ------------------------------------------------------------------ in 64 bits
def _bf16(v):
    return v.to(torch.float32).to(torch.bfloat16).to(torch.float64)


def _exact_z(x):
    """Normalised series of x [n_time][n_sub][pixels] as [pixels][n_sub][n_time] in FP64."""
    v = x.permute(2, 1, 0).to(torch.float32).contiguous()
    n = v.shape[-1]
    o = v.sort(dim=-1).values.double()
    med = (o[..., (n - 1) // 2] + o[..., n // 2]) * 0.5
    v = v.double() - med[..., None]
    o = v.abs().sort(dim=-1).values
    sig = 1.482602218505602 * (o[..., (n - 1) // 2] + o[..., n // 2]) * 0.5
    return torch.where(sig[..., None] > 0, v / sig[..., None], torch.zeros_like(v))


def _exact_maps(z, dms, widths, dt_ms):
    """S/N maxima [n_dm][n_width][pixels] of normalised series z [pixels][n_sub][n_time] in FP64."""
    npix, ns, nt = z.shape
    f = _freqs(ns)
    out = torch.full((len(dms), len(widths), npix), -math.inf, dtype=torch.float64, device=z.device)
    for d, dm in enumerate(dms):
        off = synth.arrival_offsets(dm, f, f.max(), dt_ms)
        length = nt - int(off.max())
        if length < 1:
            continue
        acc = torch.zeros((npix, length + 1), dtype=torch.float64, device=z.device)
        for s in range(ns):
            acc[:, 1:] += z[:, s, int(off[s]):int(off[s]) + length]
        acc = acc.cumsum(dim=1)
        for k, w in enumerate(widths):
            if w <= length:
                out[d, k] = (acc[:, w:] - acc[:, :-w]).max(dim=1).values / math.sqrt(ns * w)
    return out


def _exact_search(x, dms, widths, dt_ms, normalised=False):
    npix = x.shape[0] if normalised else x.shape[2]
    step = max(1, (1 << 25) // (x.numel() // npix))
    out = []
    for p in range(0, npix, step):
        z = x[p:p + step].double() if normalised else _exact_z(x[:, :, p:p + step])
        out.append(_exact_maps(z, dms, widths, dt_ms))
    return torch.cat(out, dim=2)


def _bin(x, f):
    n = x.shape[0] // f
    return x[:n * f].double().reshape(n, f, x.shape[1], x.shape[2]).sum(dim=1)


def _conv(a, w, flip=False):
    """'same' 3x3x3 convolution of a [n][t][y][x][c] with w [out][27][c] in FP64."""
    t, y, x = a.shape[1:4]
    p = torch.nn.functional.pad(a, (0, 0, 1, 1, 1, 1, 1, 1))
    out = None
    for tap in range(27):
        dt, dy, dx = tap // 9, tap // 3 % 3, tap % 3
        v = p[:, dt:dt + t, dy:dy + y, dx:dx + x].reshape(-1, a.shape[-1]) @ w[:, 26 - tap if flip else tap].T
        out = v if out is None else out.add_(v)
    return out.reshape(*a.shape[:4], w.shape[0])


def _conv_grad(a, g):
    """Weight gradient [out][27][c] of that convolution for the output gradient g."""
    t, y, x = a.shape[1:4]
    p = torch.nn.functional.pad(a, (0, 0, 1, 1, 1, 1, 1, 1))
    gm = g.reshape(-1, g.shape[-1]).T.contiguous()
    return torch.stack([gm @ p[:, k // 9:k // 9 + t, k // 3 % 3:k // 3 % 3 + y, k % 3:k % 3 + x].reshape(-1, a.shape[-1])
                        for k in range(27)], dim=1)


def _exact_network(case, seed, train):
    """Forward (and backward) pass in FP64; activations and gradients are rounded to BF16 where the network stores them."""
    x, labels = _cutout_batch(case, seed)
    th = torch.from_numpy(_parameters(seed)).cuda().double()
    ws, bs, at = [], [], 0
    for cin in CONV_IN:
        ws.append(_bf16(th[at:at + 32 * 27 * cin].reshape(32, 27, cin)))
        at += 32 * 27 * cin
        bs.append(th[at:at + 32])
        at += 32
    w1, c1, w2, c2 = th[at:at + 2048].reshape(32, 64), th[at + 2048:at + 2080], th[at + 2080:at + 2112], th[at + 2112]
    acts = [x.double()]
    for w, b in zip(ws, bs):
        acts.append(_bf16(torch.relu(_conv(acts[-1], w) + b)))
    n = case["n"]
    flat = acts[4].reshape(n, -1, 32)
    centre = ((case["t"] // 2) * case["ny"] + case["ny"] // 2) * 32 + 16
    top = flat.max(dim=1)
    arg = (flat == top.values[:, None]).to(torch.uint8).argmax(dim=1)        # the first position on ties
    h = torch.cat([top.values, flat[:, centre]], dim=1)
    u = h @ w1.T + c1
    z = torch.relu(u) @ w2 + c2
    prob = torch.sigmoid(z)
    if not train:
        return prob
    loss = torch.nn.functional.binary_cross_entropy_with_logits(z, labels.double())
    dz = (prob - labels.double()) / n
    du = torch.where(u > 0, dz[:, None] * w2, torch.zeros_like(u))
    dh = du @ w1
    g = torch.zeros_like(flat)
    g.scatter_(1, arg[:, None], dh[:, None, :32])
    g[:, centre] += dh[:, 32:]
    g = _bf16(torch.where(flat > 0, g, torch.zeros_like(g))).reshape(acts[4].shape)
    head = [(du.T @ h).reshape(-1), du.sum(dim=0), (dz[:, None] * torch.relu(u)).sum(dim=0), dz.sum().reshape(1)]
    parts = []
    for layer in range(3, -1, -1):
        parts = [_conv_grad(acts[layer], g).reshape(-1), g.reshape(-1, 32).sum(dim=0)] + parts
        if layer:
            g = _conv(g, ws[layer].permute(2, 1, 0).contiguous(), flip=True)
            g = _bf16(torch.where(acts[layer] > 0, g, torch.zeros_like(g)))
    return {"loss": loss.reshape(()), "grads": torch.cat(parts + head)}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("search", "stream", "multiscale") and case["nx"] * case["ny"] * case["n_sub"] * case["n_time"] > 1 << 30:
        return None                                   # over 20 seconds
    if kind == "search":
        x = _sky(case, case["n_time"], seed, TORCH[case["raw"]])
        return {"snr": _exact_search(x, _dms(case), _widths(case), DT_MS)}
    if kind == "stream":
        n_fill, x = _stream_chunks(case, seed)
        end = (n_fill + 1) * case["chunk"]
        return {"snr": _exact_search(x[end - case["n_time"]:end], _dms(case), _widths(case), DT_MS)}
    if kind == "multiscale":
        x = _sky(case, case["n_time"], seed, torch.float32)
        dms, widths = _dms(case), _widths(case)
        return {"snr": [_exact_search(x, dms, widths, DT_MS), _exact_search(_bin(x, 5), dms * 5.0, widths, DT_MS * 5),
                        _exact_search(_bin(x, 75), np.zeros(1), widths, DT_MS * 75)]}
    if kind == "batch":
        out = []
        for i, c in enumerate(_batch_cases(case)):
            m = _exact_search(_batch_cube(case, c, i, seed), _dms(c), _widths(c), DT_MS, case["layout"] == "pst")
            out.append({"snr": m.reshape(-1, m.shape[-1]).max(dim=0).values})
        return out
    if kind == "cutouts":
        c, desc = _cutout_plan(case, seed)
        side, nt = case["side"], case["n_time"]
        out = torch.zeros((case["n"], 64, 32, 32, 16), dtype=torch.float64, device="cuda")
        cubes = _cutout_cubes(case, seed)
        f = _freqs(16)
        for k, (cube, px, py, dm, toa) in enumerate(desc):
            off = synth.arrival_offsets(_dms(c)[dm], f, f.max(), DT_MS)
            z = cubes[cube].reshape(side, side, 16, nt)
            x0, x1, y0, y1 = max(0, px - 16), min(side, px + 16), max(0, py - 16), min(side, py + 16)
            for s in range(16):
                t = toa - 32 + int(off[s])
                a, b = max(0, t), min(nt, t + 64)
                if b > a:
                    out[k, a - t:b - t, y0 - py + 16:y1 - py + 16, x0 - px + 16:x1 - px + 16, s] = \
                        z[y0:y1, x0:x1, s, a:b].permute(2, 0, 1).double()
        return out
    return _exact_network(case, seed, kind == "train")
