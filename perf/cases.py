"""The calls a user of this library makes, as cases that can be timed and checked.

Each case is one pass through the public Python entry points (``binding.sys_conv1d`` and its
strided and 2-D relatives).  A pass is one call, except for the separable filter, which is a row
pass followed by a column pass with the intermediate image in the caller's hands.

What a user's program has before the call: the signal or image on the device, the taps as a numpy
array on the host, and (``"out": "given"``) the output tensor of a buffer that is used again and
again; with ``"out": "new"`` the call makes the output, as in examples/quickstart.py.

Signals are uniform on [-1, 1], images uniform on [0, top) with ``top`` 1 (normalised images) or 255
(grey levels as they come from a camera), taps uniform on [-1, 1]: the distributions of the benchmark workloads.
BSM, FSM, FFS and the generic kernel are not here: they reproduce the ranking of the paper's designs
and are not meant to serve.
"""
import math

import numpy as np
import torch

from paper_2010_15884_amd import binding

LARGEST_SIGNAL = 1 << 26
LARGEST_IMAGE = 8192 * 8192


def _signal(name, n, k, stride=1, projection="AUTO", out="given"):
    c = {"kind": "signal", "n": n, "k": k, "stride": stride, "projection": projection, "out": out}
    return dict(c, name=name) if name else c


def _image(name, h, w, kh, kw, stride=1, projection="AUTO", out="given", top=1.0, pad=0):
    c = {"kind": "image", "h": h, "w": w, "kh": kh, "kw": kw, "stride": stride, "projection": projection,
         "out": out, "top": top, "pad": pad}
    return dict(c, name=name) if name else c


def _separable(name, h, w, kh, kw, top=1.0):
    c = {"kind": "separable", "h": h, "w": w, "kh": kh, "kw": kw, "top": top}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a short signal, one call of a chain of small ones: launch and host time
        _signal("signal_64k_k5", 65536, 5, out="new"),
        # the headline workload: a long recording through a 16-tap filter
        _signal("signal_64m_k16", 1 << 26, 16),
        # a sharp band-pass, near the longest filter there is, on a recording of odd length
        _signal("signal_20m_k63", 20_000_003, 63),
        # a decimating half-band filter: every second output
        _signal("signal_48m_k31_s2", 48_000_001, 31, stride=2),
        # a small image through an edge filter: the smallest 2-D call in earnest
        _image("image_1k_3x3", 1024, 1024, 3, 3, out="new"),
        # the usual smoothing filter on a large image
        _image("image_4k_5x5", 4096, 4096, 5, 5),
        # a large filter on the largest image
        _image("image_8k_11x11", 8192, 8192, 11, 11),
        # the same for a caller that can promise |x| < 8 and asks for the matrix cores
        _image("image_8k_11x11_mfma", 8192, 8192, 11, 11, projection="MFMA"),
        # the largest filter, on a photograph of odd sides with grey levels 0 .. 255
        _image("image_3001x4003_15x15", 3001, 4003, 15, 15, top=255.0),
        # a separable filter as its two passes
        _separable("separable_4k_5x5", 4096, 4096, 5, 5),
        # the paper's experiment at stride 2
        _image("image_8k_5x5_s2", 8192, 8192, 5, 5, stride=2),
        # halving a ragged image through a larger filter (the first layer of an image pyramid)
        _image("image_4095x6001_7x7_s2", 4095, 6001, 7, 7, stride=2),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["signal", "signal", "image", "image", "image", "halved", "halved_signal", "mfma", "separable"])
    if kind in ("signal", "halved_signal"):
        n, k = _log_int(rng, 1 << 16, LARGEST_SIGNAL), _log_int(rng, 2, 64)
        if kind == "halved_signal":
            return _signal(None, n, k, stride=2)
        return _signal(None, n, k, projection=rng.choice(["AUTO", "AUTO", "AUTO", "AUTO", "FBS", "BFS", "SBM"]))
    h = _log_int(rng, 256, 8192)
    w = _log_int(rng, 256, 8192)
    if rng.random() < 0.3:
        w = h                                            # square ones are common
    if kind == "separable":
        return _separable(None, h, w, rng.randint(2, 15), rng.randint(2, 15), top=rng.choice([1.0, 255.0]))
    largest = 13 if kind == "mfma" else 15
    kh = rng.randint(2, largest)
    kw = kh if rng.random() < 0.7 else rng.randint(1, largest)      # most filters are square
    while h * w * kh * kw > LARGEST_IMAGE * 121:                    # no dearer than the largest listed case
        h, w = max(256, h * 3 // 4), max(256, w * 3 // 4)
    pad = rng.choice([0, 0, 0, rng.randint(1, 64)])                 # a region of a wider image
    top = rng.choice([1.0, 1.0, 255.0])
    if kind == "mfma":
        return _image(None, h, w, kh, kw, projection="MFMA", pad=pad)
    if kind == "halved":
        return _image(None, h, w, kh, kw, stride=2, top=top, pad=pad)
    projection = "AUTO"
    if rng.random() < 0.25:
        projection = rng.choice(["FBS", "BFS", "SBM"] if kh == kw and kh <= 11 else ["FBS"])
    return _image(None, h, w, kh, kw, projection=projection, top=top, pad=pad)


def _out_shape(case):
    if case["kind"] == "signal":
        return ((case["n"] - case["k"]) // case["stride"] + 1,)
    s = case.get("stride", 1)
    return ((case["h"] - case["kh"]) // s + 1, (case["w"] - case["kw"]) // s + 1)


def _inputs(case, seed):
    """The device input and the host taps (one array, or two for the separable filter)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    taps = np.random.default_rng(int(seed))
    if case["kind"] == "signal":
        x = torch.empty(case["n"], dtype=torch.float32, device="cuda").uniform_(-1.0, 1.0, generator=gen)
        return x, taps.uniform(-1.0, 1.0, case["k"]).astype(np.float32)
    pad = case.get("pad", 0)
    x = torch.empty((case["h"], case["w"] + pad), dtype=torch.float32, device="cuda")
    x = x.uniform_(0.0, case["top"], generator=gen)[:, :case["w"]]
    if case["kind"] == "separable":
        return x, (taps.uniform(-1.0, 1.0, (1, case["kw"])).astype(np.float32),
                   taps.uniform(-1.0, 1.0, (case["kh"], 1)).astype(np.float32))
    return x, taps.uniform(-1.0, 1.0, (case["kh"], case["kw"])).astype(np.float32)


def prepare(case, seed):
    x, taps = _inputs(case, seed)
    state = {"case": case, "x": x, "taps": taps, "y": None}
    if case["kind"] == "separable":
        # intermediate rows on 128-byte lines, as the library's documentation advises
        ow = case["w"] - case["kw"] + 1
        state["mid"] = torch.empty((case["h"], (ow + 31) // 32 * 32), dtype=torch.float32, device="cuda")[:, :ow]
        state["y"] = torch.empty(_out_shape(case), dtype=torch.float32, device="cuda")
    elif case["out"] == "given":
        state["y"] = torch.empty(_out_shape(case), dtype=torch.float32, device="cuda")
    return state


def run(state):
    case, x, taps, y = state["case"], state["x"], state["taps"], state["y"]
    if case["kind"] == "separable":
        row, column = taps
        binding.sys_conv2d(x, row, state["mid"])
        return binding.sys_conv2d(state["mid"], column, y)
    if case["kind"] == "signal":
        if case["stride"] == 1:
            return binding.sys_conv1d(x, taps, y, projection=case["projection"])
        return binding.sys_conv1d_strided(x, taps, case["stride"], y, projection=case["projection"])
    if case["stride"] == 1:
        return binding.sys_conv2d(x, taps, y, projection=case["projection"])
    return binding.sys_conv2d_strided(x, taps, case["stride"], y, projection=case["projection"])


def work(case):
    outputs = math.prod(_out_shape(case))
    if case["kind"] == "signal":
        return {"bytes": 4 * (case["n"] + outputs + case["k"]), "flops": 2 * case["k"] * outputs}
    inputs = case["h"] * case["w"]
    if case["kind"] == "separable":
        mid = case["h"] * (case["w"] - case["kw"] + 1)
        # two calls: the intermediate image is written by one and read by the other
        return {"bytes": 4 * (inputs + 2 * mid + outputs + case["kh"] + case["kw"]),
                "flops": 2 * (case["kw"] * mid + case["kh"] * outputs)}
    taps = case["kh"] * case["kw"]
    return {"bytes": 4 * (inputs + outputs + taps), "flops": 2 * taps * outputs}


def tolerance(case):
    # All sums are fp32.  Against the 64-bit definition every projection (each has an order of its own)
    # is off by 4e-8 .. 2.9e-7 (2-norm) and by at most 2.6e-6 (largest difference over the root mean
    # square) on the listed cases and 16 drawn ones, more with the number of taps and where the taps
    # happen to cancel the mean of the image; the bounds are about four times the worst of that.
    return {"rel": 2e-6, "max": 1.5e-5}


def exact(case, seed):
    """The definition in 64 bits: one shifted slice of the input per tap."""
    x, taps = _inputs(case, seed)
    x = x.double()
    if case["kind"] == "separable":
        row, column = taps
        return _sum_2d(_sum_2d(x, row, 1), column, 1)
    if case["kind"] == "signal":
        n, k, s = case["n"], case["k"], case["stride"]
        m = _out_shape(case)[0]
        y = torch.zeros(m, dtype=torch.float64, device=x.device)
        for q in range(k):
            y.add_(x[q:q + s * (m - 1) + 1:s], alpha=float(taps[q]))
        return y
    return _sum_2d(x, taps, case["stride"])


def _sum_2d(x, f, s):
    oh, ow = (x.shape[0] - f.shape[0]) // s + 1, (x.shape[1] - f.shape[1]) // s + 1
    y = torch.zeros((oh, ow), dtype=torch.float64, device=x.device)
    for p in range(f.shape[0]):
        for q in range(f.shape[1]):
            y.add_(x[p:p + s * (oh - 1) + 1:s, q:q + s * (ow - 1) + 1:s], alpha=float(f[p, q]))
    return y
