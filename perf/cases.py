"""Performance cases of the library: the calls a user's program makes, over the sizes it makes them at.

`listed()` names twelve calls, `draw(rng)` gives one more of the same ranges.  A case says which entry point is called
and with what shapes; `prepare` makes what the program holds before the call (tensors, workspace, result tensor),
`run` makes the call once, `work` is what it cannot do without, `exact` its result in 64 bits by plain torch.
"""
import math

import torch

from paper_1606_05688_amd import binding as znni

DEVICE = "cuda"


def _layer(entry, S, f, fo, n, k, bias=True, relu=True):
    n = (n,) * 3 if isinstance(n, int) else tuple(n)
    k = (k,) * 3 if isinstance(k, int) else tuple(k)
    return {"entry": entry, "S": S, "f": f, "fo": fo, "nx": n[0], "ny": n[1], "nz": n[2],
            "kx": k[0], "ky": k[1], "kz": k[2], "bias": bias, "relu": relu}


def _pool(entry, S, f, n, p):
    n = (n,) * 3 if isinstance(n, int) else tuple(n)
    p = (p,) * 3 if isinstance(p, int) else tuple(p)
    return {"entry": entry, "S": S, "f": f, "nx": n[0], "ny": n[1], "nz": n[2], "px": p[0], "py": p[1], "pz": p[2]}


# entry: what the program calls
#   "choose"  znni_conv3d: the library picks the primitive, result and workspace come from torch's allocator
#   "fft"     znni_conv3d_fft on a result tensor and a workspace that the program keeps
#   "kept"    the same with keep_kernels: one kernel bank meets many patches, its transforms are kept in the workspace
#   "static"  znni_conv3d_fft_static: the entry point for programs that may not allocate
#   "budget"  znni_conv3d_fft_budget on half of the workspace the whole layer would take
#   "mpf" / "maxpool"  the pooling layers
def listed():
    return [
        # the smallest layer anyone runs: launches and host time only (the first benchmark layer)
        {"name": "tiny_2to3_16_k3", **_layer("fft", 1, 2, 3, 16, 3, bias=False, relu=False)},
        # a narrow layer on a small patch in a serving loop that may not allocate (the second benchmark layer)
        {"name": "static_8to8_64_k5", **_layer("static", 1, 8, 8, 64, 5)},
        # a wide layer of small kernels on a medium patch (the third benchmark layer), primitive left to the library
        {"name": "wide_40to40_128_k3", **_layer("choose", 1, 40, 40, 128, 3)},
        # a layer behind one pooling layer: a batch of fragments (the fourth benchmark layer)
        {"name": "batch_8x32to32_64_k7", **_layer("fft", 8, 32, 32, 64, 7)},
        # an early layer on a whole sub-volume (the fifth and largest benchmark layer)
        {"name": "large_48to48_320_k5", **_layer("fft", 1, 48, 48, 320, 5)},
        # first layer of a network: one grey image in, many feature maps out
        {"name": "first_1to48_128_k3", **_layer("choose", 1, 1, 48, 128, 3)},
        # few maps in, many out, smallest kernels: where convolving directly pays
        {"name": "narrow_8to80_200_k2", **_layer("choose", 1, 8, 80, 200, 2)},
        # a layer behind two pooling layers: many small fragments, one bank for all patches of a volume
        {"name": "kept_64x80to80_51_k5", **_layer("kept", 64, 80, 80, 51, 5)},
        # a wide layer of large kernels, one bank for all patches of a volume
        {"name": "kept_80to80_128_k7", **_layer("kept", 1, 80, 80, 128, 7)},
        # sizes nobody chose for speed: odd edges that differ by axis, anisotropic kernels (as for EM stacks), no
        # multiple of any tile
        {"name": "ragged_37to45_93x110x131", **_layer("choose", 1, 37, 45, (93, 110, 131), (3, 4, 5))},
        # a layer that has to make do with half of the memory it would like
        {"name": "budget_48to48_160_k5", **_layer("budget", 1, 48, 48, 160, 5)},
        # the pooling layer that makes the fragments
        {"name": "mpf_48_255_p2", **_pool("mpf", 1, 48, 255, 2)},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _bytes(c):
    return work(c)["bytes"]


def draw(rng):
    """One more call of the ranges that the listed ones span; never dearer than the largest of them."""
    most = 3.0e9
    while True:
        kind = rng.choice(("choose", "choose", "fft", "fft", "batch", "batch", "first", "kept", "static", "budget", "mpf",
                           "maxpool"))
        cubic = rng.random() < 0.5
        if kind in ("mpf", "maxpool"):
            p = [rng.choice((1, 2, 2, 2, 3, 4)) for _ in range(3)] if not cubic else [rng.choice((2, 2, 3, 4))] * 3
            e = [_log_int(rng, 20, 300) for _ in range(3)] if not cubic else [_log_int(rng, 20, 300)] * 3
            add = -1 if kind == "mpf" else 0
            n = [max(2 * q, v // q * q) + (add if q > 1 else 0) for v, q in zip(e, p)]
            c = _pool(kind, _log_int(rng, 1, 8), _log_int(rng, 1, 96), n, p)
            if _bytes(c) <= most:
                return c
            continue
        k = [rng.randint(2, 7)] * 3 if cubic else [rng.randint(1, 7) for _ in range(3)]
        S = _log_int(rng, 2, 64) if kind == "batch" else (rng.choice((1, 1, 1, 8, 27)) if kind == "kept" else 1)
        top = {"batch": 100, "static": 64, "kept": 160 if S == 1 else 64}.get(kind, 320)
        base = _log_int(rng, 12 if kind in ("fft", "static") else 24, top)
        n = [base] * 3 if cubic else [max(q, int(base * rng.uniform(0.7, 1.4))) for q in k]
        if kind == "first":
            S, f, fo = 1, rng.randint(1, 8), _log_int(rng, 16, 96)
            k = [min(q, 4) for q in k]
            kind = "choose"
        elif kind == "static":
            f, fo = rng.randint(1, 12), rng.randint(1, 12)
        else:
            f, fo = _log_int(rng, 4, 96), _log_int(rng, 4, 96)
        c = _layer("fft" if kind == "batch" else kind, S, f, fo, n, k, bias=rng.random() < 0.8, relu=rng.random() < 0.8)
        if _bytes(c) > most or 2.0 * f * fo * S * n[0] * n[1] * n[2] > 6.0e11:
            continue
        if kind == "static" and znni.znni_conv3d_fft_workspace(S, f, fo, tuple(n), tuple(k)) > znni.STATIC_SCRATCH_BYTES:
            continue
        return c


def _shape(c):
    return (c["nx"], c["ny"], c["nz"]), (c["kx"], c["ky"], c["kz"])


def prepare(case, seed):
    c = case
    g = torch.Generator(device=DEVICE).manual_seed(int(seed))
    n = (c["nx"], c["ny"], c["nz"])
    inp = torch.empty((c["S"], c["f"]) + n, dtype=torch.float32, device=DEVICE).uniform_(-1.0, 1.0, generator=g)
    if c["entry"] in ("mpf", "maxpool"):
        p = (c["px"], c["py"], c["pz"])
        frag = p[0] * p[1] * p[2] if c["entry"] == "mpf" else 1
        out = torch.empty((c["S"] * frag, c["f"]) + tuple(a // b for a, b in zip(n, p)), dtype=torch.float32, device=DEVICE)
        return {"case": dict(c), "inp": inp, "p": p, "out": out}
    n, k = _shape(c)
    std = (c["f"] * k[0] * k[1] * k[2]) ** -0.5
    w = torch.empty((c["fo"], c["f"]) + k, dtype=torch.float32, device=DEVICE).normal_(0.0, std, generator=g)
    bias = None
    if c["bias"]:
        bias = torch.empty((c["fo"],), dtype=torch.float32, device=DEVICE).normal_(0.0, 0.1 ** 0.5, generator=g)
    st = {"case": dict(c), "inp": inp, "w": w, "bias": bias, "relu": c["relu"]}
    if c["entry"] == "choose":
        return st
    st["out"] = torch.empty((c["S"], c["fo"]) + tuple(a - b + 1 for a, b in zip(n, k)), dtype=torch.float32, device=DEVICE)
    if c["entry"] in ("fft", "kept"):
        st["workspace"] = znni.alloc_workspace(c["S"], c["f"], c["fo"], n, k)
    if c["entry"] == "budget":
        half = znni.znni_conv3d_fft_workspace(c["S"], c["f"], c["fo"], n, k) // 2
        st["workspace"] = torch.empty(half, dtype=torch.uint8, device=DEVICE)
    if c["entry"] == "kept":
        # the first patch of the volume: stores the kernel bank's transforms in the workspace
        znni.znni_conv3d_fft(inp, w, bias, relu=c["relu"], out=st["out"], workspace=st["workspace"])
    return st


def run(state):
    s = state
    entry = s["case"]["entry"]
    if entry == "choose":
        return znni.znni_conv3d(s["inp"], s["w"], s["bias"], relu=s["relu"])
    if entry == "fft":
        return znni.znni_conv3d_fft(s["inp"], s["w"], s["bias"], relu=s["relu"], out=s["out"], workspace=s["workspace"])
    if entry == "kept":
        return znni.znni_conv3d_fft(s["inp"], s["w"], s["bias"], relu=s["relu"], out=s["out"], workspace=s["workspace"],
                                    keep_kernels=True)
    if entry == "static":
        return znni.znni_conv3d_fft_static(s["inp"], s["w"], s["bias"], relu=s["relu"], out=s["out"])
    if entry == "budget":
        return znni.znni_conv3d_fft_budget(s["inp"], s["w"], s["bias"], relu=s["relu"], out=s["out"],
                                           workspace=s["workspace"])
    if entry == "mpf":
        return znni.znni_mpf(s["inp"], s["p"], out=s["out"])
    return znni.znni_maxpool(s["inp"], s["p"], out=s["out"])


def work(case):
    """Bytes: image, kernels and bias in, result out.  Flops: the cheaper of the direct sum and one transform of every
    image at its own size (2.5 N log2 N each) with the products of the halved spectra (8 per complex multiply-add)."""
    c = case
    vox = c["nx"] * c["ny"] * c["nz"]
    if c["entry"] in ("mpf", "maxpool"):
        p = (c["px"], c["py"], c["pz"])
        m = math.prod(a // b for a, b in zip((c["nx"], c["ny"], c["nz"]), p))
        pv = math.prod(p)
        frag = pv if c["entry"] == "mpf" else 1
        outs = c["S"] * c["f"] * frag * m
        return {"bytes": 4 * (c["S"] * c["f"] * vox + outs), "flops": outs * max(pv - 1, 1)}
    n, k = _shape(c)
    ovox, kv = math.prod(a - b + 1 for a, b in zip(n, k)), math.prod(k)
    nbytes = 4 * (c["S"] * c["f"] * vox + c["f"] * c["fo"] * kv + (c["fo"] if c["bias"] else 0) + c["S"] * c["fo"] * ovox)
    direct = 2.0 * c["S"] * c["f"] * c["fo"] * kv * ovox
    fft = 2.5 * c["S"] * (c["f"] + c["fo"]) * vox * math.log2(max(vox, 2)) + 4.0 * c["S"] * c["f"] * c["fo"] * vox
    return {"bytes": nbytes, "flops": min(direct, fft)}


def tolerance(case):
    if case["entry"] in ("mpf", "maxpool"):
        return "exact"
    # 32-bit transforms and sums: 1e-7 to 6e-7 off the 64-bit result, so two correct implementations are up to 8e-7 apart
    return {"rel": 3e-6, "max": 3e-5}


def exact(case, seed):
    """The layer as its definition has it, summed tap by tap in 64 bits (kernel flipped, valid outputs only)."""
    c = case
    if c["entry"] in ("mpf", "maxpool"):
        s = prepare(case, seed)
        x, p = s["inp"].double(), s["p"]
        if c["entry"] == "maxpool":
            return torch.nn.functional.max_pool3d(x, p)
        m = [a // b for a, b in zip(x.shape[2:], p)]
        res = torch.empty(s["out"].shape, dtype=torch.float64, device=DEVICE)
        pv = p[0] * p[1] * p[2]
        for ox in range(p[0]):
            for oy in range(p[1]):
                for oz in range(p[2]):
                    y = x[:, :, ox:ox + m[0] * p[0], oy:oy + m[1] * p[1], oz:oz + m[2] * p[2]].contiguous()
                    res[(ox * p[1] + oy) * p[2] + oz::pv] = torch.nn.functional.max_pool3d(y, p)
        return res
    s = prepare({**case, "entry": "choose"}, seed)
    n, k = _shape(c)
    o = [a - b + 1 for a, b in zip(n, k)]
    if c["S"] * c["f"] * c["fo"] * math.prod(o) * math.prod(k) > 2.0e13:
        return None
    wd = s["w"].double()
    res = torch.empty((c["S"], c["fo"]) + tuple(o), dtype=torch.float64, device=DEVICE)
    xd = torch.empty((c["f"], n[0], n[1], n[2]), dtype=torch.float64, device=DEVICE)
    for q in range(c["S"]):
        xd.copy_(s["inp"][q])
        acc = torch.zeros((c["fo"], math.prod(o)), dtype=torch.float64, device=DEVICE)
        for a in range(k[0]):
            for b in range(k[1]):
                for e in range(k[2]):
                    x0, y0, z0 = k[0] - 1 - a, k[1] - 1 - b, k[2] - 1 - e
                    sl = xd[:, x0:x0 + o[0], y0:y0 + o[1], z0:z0 + o[2]].contiguous().view(c["f"], -1)
                    acc.addmm_(wd[:, :, a, b, e].contiguous(), sl)
        res[q] = acc.view(c["fo"], *o)
    if s["bias"] is not None:
        res += s["bias"].double().view(1, -1, 1, 1, 1)
    if c["relu"]:
        res.clamp_(min=0.0)
    return res
