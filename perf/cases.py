"""The work that users of this library have it do, as cases that can be timed
and compared: image filters, edge maps and the 8-bit image pipeline, ragged
batches, the separable filter, and filter banks (convolution layers) forward
and backward in FP32 and BF16.

A case is a dict of plain values.  ``listed()`` gives the standing cases,
``draw(rng)`` one more of the same ranges, ``prepare`` what a program holds
before the call, ``run`` one pass through the public entry points, ``work``
the bytes and operations of a pass, and ``exact`` the results in 64 bits,
computed with plain torch operations only.
"""
import math

import torch

from paper_2504_01266_amd import binding
from paper_2504_01266_amd.autograd import filter2d

LAPLACIAN = [[-1.0, -1.0, -1.0], [-1.0, 8.0, -1.0], [-1.0, -1.0, -1.0]]
SOBEL_X = [[-1, 0, 1], [-2, 0, 2], [-1, 0, 1]]
GRAY_RGB = [0.299, 0.587, 0.114]

# a drawn case costs no more than the listed FP32 training step
MAX_DRAWN_BYTES = 7.0e9
MAX_DRAWN_FLOPS = 9.0e11


def listed():
    return [
        # a single small patch, as an interactive tool or a unit of a tiled
        # program filters it: launch latency
        {"name": "patch", "kind": "filter", "n": 1, "c": 3, "h": 64, "w": 64, "k": 5, "border": "clamp"},
        # one grayscale image, the 5x5 Gaussian blur
        {"name": "blur", "kind": "filter", "n": 1, "c": 1, "h": 1024, "w": 1024, "k": 5, "border": "clamp"},
        # the sharpen of a 4K frame held in FP32 (out-of-image neighbours skipped)
        {"name": "sharpen_4k", "kind": "filter", "n": 1, "c": 3, "h": 2160, "w": 3840, "k": 3, "border": "zero"},
        # edge maps of an 8K 8-bit frame: Sobel x, Sobel y and their squared magnitude
        {"name": "sobel_8k", "kind": "edges", "n": 1, "c": 3, "h": 4320, "w": 7680},
        # upsample then sharpen of an interleaved 8-bit 4K frame, as OpenCV delivers it
        {"name": "upsharpen_4k", "kind": "upsharpen", "n": 1, "c": 3, "h": 2160, "w": 3840, "scale": 2},
        # grayscale of an interleaved 8-bit 8K frame
        {"name": "gray_8k", "kind": "gray", "n": 1, "c": 3, "h": 4320, "w": 7680},
        # a batch of images through a separable 9x9 Gaussian
        {"name": "separable", "kind": "separable", "n": 16, "c": 3, "h": 2048, "w": 2048, "k": 9},
        # a batch of photographs of all sizes, each with its own 7x7 filter
        {"name": "ragged", "kind": "ragged", "items": 64, "lo": 256, "hi": 4096, "c": 3, "k": 7, "sizes": 3},
        # learning one shared 9x9 filter: forward and both gradients
        {"name": "train_shared", "kind": "train", "mode": "shared", "dtype": "f32", "n": 16, "ci": 3, "co": 3,
         "h": 2048, "w": 2048, "k": 9},
        # a training step of an FP32 3x3 convolution layer
        {"name": "train_bank_f32", "kind": "train", "mode": "bank", "dtype": "f32", "n": 16, "ci": 16, "co": 64,
         "h": 1024, "w": 1024, "k": 3},
        # a training step of the BF16 5x5 layer, upstream gradients in BF16
        {"name": "bank_step_bf16", "kind": "bank_step", "n": 32, "ci": 16, "co": 64, "h": 1024, "w": 1024, "k": 5},
        # inference of a BF16 3x3 layer on images of odd sizes, BF16 activations out
        {"name": "bank_infer_odd", "kind": "bank_infer", "n": 8, "ci": 16, "co": 64, "h": 509, "w": 763, "k": 3},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _drawn(rng):
    kind = rng.choice(["filter", "filter", "edges", "upsharpen", "gray", "separable", "ragged", "train", "train",
                       "bank_step", "bank_infer"])
    h, w = _log_int(rng, 33, 4320), _log_int(rng, 33, 7680)
    if kind == "filter":
        return {"kind": kind, "n": rng.choice([1, 1, 2, 5]), "c": rng.choice([1, 3, 4]), "h": h, "w": w,
                "k": rng.choice([3, 5, 7, 9]), "border": rng.choice(["clamp", "zero"])}
    if kind in ("edges", "gray"):
        return {"kind": kind, "n": rng.choice([1, 1, 3]), "c": 3, "h": h, "w": w}
    if kind == "upsharpen":
        return {"kind": kind, "n": 1, "c": rng.choice([3, 3, 4]), "h": min(h, 2160), "w": min(w, 3840),
                "scale": rng.choice([1, 2, 3, 4, 5])}
    if kind == "separable":
        return {"kind": kind, "n": rng.choice([1, 4, 16]), "c": rng.choice([1, 3]), "h": min(h, 2048),
                "w": min(w, 2048), "k": rng.choice([3, 5, 7, 9, 11, 15])}
    if kind == "ragged":
        lo = _log_int(rng, 16, 256)
        return {"kind": kind, "items": rng.randint(2, 48), "lo": lo, "hi": _log_int(rng, 2 * lo, 4096),
                "c": rng.choice([1, 3]), "k": rng.choice([3, 5, 7, 9]), "sizes": rng.randint(1, 1 << 20)}
    if kind == "train" and rng.random() < 0.5:
        return {"kind": kind, "mode": "shared", "dtype": "f32", "n": rng.choice([1, 4, 16]), "ci": 3, "co": 3,
                "h": min(h, 2048), "w": min(w, 2048), "k": rng.choice([3, 5, 7, 9])}
    n, k = rng.choice([1, 2, 4, 8]), rng.choice([1, 3, 3, 5])
    ci, co = rng.choice([(3, 16), (8, 16), (16, 16), (16, 32), (16, 64), (12, 24), (32, 64), (64, 64), (64, 16)])
    dtype = rng.choice(["f32", "f32", "bf16"])
    if kind == "bank_step" or kind == "train" and dtype == "bf16":
        ci = min(ci, 16)  # what the BF16 backward takes
    h, w = _log_int(rng, 28, 1024), _log_int(rng, 28, 1024)
    if rng.random() < 0.5:  # the sizes of most layers
        w = (w + 7) // 8 * 8
    if kind == "train":
        return {"kind": kind, "mode": "bank", "dtype": dtype, "n": n, "ci": ci, "co": co, "h": h,
                "w": w, "k": k}
    return {"kind": kind, "n": n, "ci": ci, "co": co, "h": h, "w": w, "k": k}


def draw(rng):
    """One more case: sizes over the whole range (33 up to an 8K frame for
    images, 28 to 1024 for layers, 16 to 4096 for ragged batches), odd ones
    among them, every kernel size and channel count that is in use."""
    while True:
        case = _drawn(rng)
        w = work(case)
        if w["bytes"] <= MAX_DRAWN_BYTES and w["flops"] <= MAX_DRAWN_FLOPS:
            return case


# ------------------------------------------------------------------ inputs --


def _gauss(k, sigma):
    d = torch.arange(k, dtype=torch.float64) - (k - 1) // 2
    g = torch.exp(-d * d / (2.0 * sigma * sigma))
    return (g / g.sum()).float()


def _ragged_sizes(case):
    gen = torch.Generator().manual_seed(case["sizes"])
    return torch.randint(case["lo"], case["hi"] + 1, (case["items"], 2), generator=gen).tolist()


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind, k = case["kind"], case.get("k", 3)

    def uniform(*shape):
        return torch.rand(shape, generator=gen, device="cuda")

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda")

    def pixels(*shape):
        return torch.randint(0, 256, shape, generator=gen, device="cuda", dtype=torch.uint8)

    st = {"case": case}
    if kind == "filter":
        st["x"] = uniform(case["n"], case["c"], case["h"], case["w"])
        g = _gauss(k, k / 5.0)
        st["f"] = (torch.tensor(LAPLACIAN) if k == 3 else torch.outer(g, g)).cuda()
    elif kind == "edges":
        st["x"] = pixels(case["n"], case["c"], case["h"], case["w"])
        sx = torch.tensor(SOBEL_X, dtype=torch.int32)
        st["f"] = torch.stack([sx, sx.t()]).repeat(case["c"], 1, 1).unsqueeze(1).contiguous().cuda()
    elif kind in ("upsharpen", "gray"):
        st["x"] = pixels(case["n"], case["h"], case["w"], case["c"]).permute(0, 3, 1, 2)
        st["f"] = (torch.tensor(LAPLACIAN) if kind == "upsharpen" else
                   torch.tensor(GRAY_RGB).view(1, 3, 1, 1)).cuda()
    elif kind == "separable":
        st["x"] = uniform(case["n"], case["c"], case["h"], case["w"])
        st["a"] = _gauss(k, k / 4.5).cuda()
    elif kind == "ragged":
        xs = [uniform(case["c"], h, w) for h, w in _ragged_sizes(case)]
        fs = [normal(k, k) / k for _ in xs]
        st["x"], st["f"], st["y"] = xs, fs, [torch.empty_like(x) for x in xs]
        st["batch"] = binding.RaggedBatch(xs, st["y"], fs)
    elif kind == "train" and case["mode"] == "shared":
        st["x"] = uniform(case["n"], case["ci"], case["h"], case["w"]).requires_grad_()
        st["f"] = (normal(k, k) / k).requires_grad_()
        st["g"] = normal(case["n"], case["co"], case["h"], case["w"])
    else:  # a filter bank
        x = normal(case["n"], case["ci"], case["h"], case["w"])
        f = normal(case["co"], case["ci"], k, k) * math.sqrt(2.0 / (case["ci"] * k * k))
        if kind != "train" or case["dtype"] == "bf16":
            x, f = x.bfloat16(), f.bfloat16()
        st["x"], st["f"] = x, f
        if kind != "bank_infer":
            g = normal(case["n"], case["co"], case["h"], case["w"])
            st["g"] = g if kind == "train" else g.bfloat16()
        if kind == "train":
            st["x"].requires_grad_()
            st["f"].requires_grad_()
    return st


# -------------------------------------------------------------------- pass --


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "filter":
        return binding.forward(st["x"], st["f"], border=case["border"])
    if kind == "edges":
        return binding.forward(st["x"], st["f"], mode="depthwise", epilogue=binding.EPI_SUMSQ_PAIRS)
    if kind == "upsharpen":
        return binding.upsample_forward(st["x"], st["f"], case["scale"], out_dtype=torch.uint8, border="zero")
    if kind == "gray":
        return binding.forward(st["x"], st["f"], mode="bank", out_dtype=torch.uint8)
    if kind == "separable":
        return binding.forward_separable(st["x"], st["a"], st["a"])
    if kind == "ragged":
        st["batch"].run()
        return st["y"]
    if kind == "train":
        x, f = st["x"], st["f"]
        x.grad = f.grad = None
        y = filter2d(x, f, case["mode"])
        y.backward(st["g"])
        return y, x.grad, f.grad
    if kind == "bank_step":
        y = binding.forward(st["x"], st["f"], mode="bank")
        return (y, *binding.backward(st["x"], st["f"], st["g"], mode="bank"))
    return binding.forward(st["x"], st["f"], mode="bank", out_dtype=torch.bfloat16)


# -------------------------------------------------------------------- work --


def work(case):
    """Bytes (each input read once, each output written once) and operations
    (two per multiply-add) of a pass; gradients that a backward reads with the
    image again count once per product."""
    kind, k = case["kind"], case.get("k", 3)
    if kind == "ragged":
        px = case["c"] * sum(h * w for h, w in _ragged_sizes(case))
        return {"bytes": 8.0 * px, "flops": 2.0 * px * k * k}
    px = case["n"] * case["h"] * case["w"]
    c = case.get("c", 1)
    if kind == "filter":
        return {"bytes": 8.0 * px * c, "flops": 2.0 * px * c * k * k}
    if kind == "edges":
        return {"bytes": 13.0 * px * c, "flops": (36.0 + 3.0) * px * c}
    if kind == "upsharpen":
        s2 = case["scale"] ** 2
        return {"bytes": 1.0 * px * c * (1 + s2), "flops": 18.0 * px * c * s2}
    if kind == "gray":
        return {"bytes": 4.0 * px, "flops": 6.0 * px}
    if kind == "separable":
        return {"bytes": 8.0 * px * c, "flops": 4.0 * px * c * k}
    ci, co = case["ci"], case["co"]
    if kind == "train" and case["mode"] == "shared":
        # forward reads X and writes Y; the backward reads G and X and writes X-bar
        return {"bytes": 4.0 * px * ci * 5, "flops": 6.0 * px * ci * k * k}
    flops = 2.0 * px * co * ci * k * k
    wts = co * ci * k * k
    if kind == "bank_infer":
        return {"bytes": 2.0 * (px * (ci + co) + wts), "flops": flops}
    if kind == "bank_step":
        # X (2 B) twice, Y (4 B), G (2 B), X-bar (4 B)
        return {"bytes": px * (8.0 * ci + 6.0 * co) + 8.0 * wts, "flops": 3.0 * flops}
    es = 4.0 if case["dtype"] == "f32" else 2.0
    # X twice, Y and G (FP32), X-bar in X's type
    return {"bytes": px * (3.0 * es * ci + 8.0 * co) + 3.0 * es * wts, "flops": 3.0 * flops}


# ------------------------------------------------------------ 64-bit values --


def _pad(x, r, border):
    """x with r more rows and columns on each side: its edge values, or zeros."""
    h, w = x.shape[-2:]
    dev = x.device
    if border == "clamp":
        iy = torch.arange(-r, h + r, device=dev).clamp(0, h - 1)
        ix = torch.arange(-r, w + r, device=dev).clamp(0, w - 1)
        return x.index_select(-2, iy).index_select(-1, ix)
    y = x.new_zeros(*x.shape[:-2], h + 2 * r, w + 2 * r)
    y[..., r:r + h, r:r + w] = x
    return y


def _fold(z, r):
    """The adjoint of _pad(..., "clamp")."""
    if r == 0:
        return z
    for dim in (-2, -1):
        n = z.shape[dim] - 2 * r
        mid = z.narrow(dim, r, n).clone()
        mid.narrow(dim, 0, 1).add_(z.narrow(dim, 0, r).sum(dim, keepdim=True))
        mid.narrow(dim, n - 1, 1).add_(z.narrow(dim, n + r, r).sum(dim, keepdim=True))
        z = mid
    return z


def _each_tap(k):
    return [(u, v) for u in range(k) for v in range(k)]


def _exact_filter(x, f, border="clamp"):
    """One [k][k] filter over every plane of x."""
    k = f.shape[-1]
    h, w = x.shape[-2:]
    xp = _pad(x.double(), (k - 1) // 2, border)
    y = torch.zeros_like(x, dtype=torch.float64)
    for u, v in _each_tap(k):
        y.add_(xp[..., u:u + h, v:v + w], alpha=float(f[u, v]))
    return y


def _exact_shared_grads(x, f, g):
    k = f.shape[-1]
    r = (k - 1) // 2
    h, w = x.shape[-2:]
    gx = torch.empty_like(x, dtype=torch.float64)
    gf = torch.zeros(k, k, dtype=torch.float64, device=x.device)
    for i in range(x.shape[0]):
        xp, gi = _pad(x[i].double(), r, "clamp"), g[i].double()
        z = gi.new_zeros(x.shape[1], h + 2 * r, w + 2 * r)
        for u, v in _each_tap(k):
            z[:, u:u + h, v:v + w].add_(gi, alpha=float(f[u, v]))
            gf[u, v] += (xp[:, u:u + h, v:v + w] * gi).sum()
        gx[i] = _fold(z, r)
    return gx, gf


def _exact_bank(x, f, g=None):
    """Forward, and both gradients where g is given, of a filter bank."""
    n, ci, h, w = x.shape
    co, k = f.shape[0], f.shape[-1]
    r = (k - 1) // 2
    fd = f.double()
    y = torch.zeros(n, co, h * w, dtype=torch.float64, device=x.device)
    gx = torch.zeros(n, ci, h, w, dtype=torch.float64, device=x.device) if g is not None else None
    gf = torch.zeros_like(fd) if g is not None else None
    for i in range(n):
        xp = _pad(x[i].double(), r, "clamp")
        gi = g[i].double().view(co, h * w) if g is not None else None
        z = x.new_zeros(ci, h + 2 * r, w + 2 * r, dtype=torch.float64) if g is not None else None
        for u, v in _each_tap(k):
            xs = xp[:, u:u + h, v:v + w].reshape(ci, h * w)
            wt = fd[:, :, u, v].contiguous()
            y[i].addmm_(wt, xs)
            if g is not None:
                z[:, u:u + h, v:v + w].add_((wt.t().contiguous() @ gi).view(ci, h, w))
                gf[:, :, u, v] += gi @ xs.t().contiguous()
        if g is not None:
            gx[i] = _fold(z, r)
    y = y.view(n, co, h, w)
    return y if g is None else (y, gx, gf)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("edges", "upsharpen", "gray"):
        return None  # whole numbers and bytes
    st = prepare(case, seed)
    with torch.no_grad():
        if kind == "filter":
            return _exact_filter(st["x"], st["f"], case["border"])
        if kind == "separable":
            a = st["a"].double()
            return _exact_filter(st["x"], torch.outer(a, a))
        if kind == "ragged":
            return [_exact_filter(x, f) for x, f in zip(st["x"], st["f"])]
        if kind == "train" and case["mode"] == "shared":
            return (_exact_filter(st["x"], st["f"]), *_exact_shared_grads(st["x"], st["f"], st["g"]))
        return _exact_bank(st["x"], st["f"], st.get("g"))
