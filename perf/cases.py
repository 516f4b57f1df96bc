"""Performance cases: what users of this package have it do, through its public entry points.

Five kinds of work:
  sample   a whole sampling run (Context.sample): refresh steps, cached steps, solver update and variance compensation
  steps    the same loop driven by the caller, one Context.sample_step at a time
  linear   quantise an activation tensor and multiply it with quantised weights (qc_quantize_act + qc_w8a8_linear)
  cluster  the calibration-set clustering of a sample pool (qc_tap_cluster)
  fit      the variance-compensation factors fitted along a trajectory (qc_vc_fit_sampler: the un-quantised reference
           network beside the quantised sampler)
Weights, latents, labels and pools are seeded draws of the real shapes, made on the GPU."""
import ctypes
import math
from types import SimpleNamespace

import torch

import paper_2503_02508_amd as qc
from paper_2503_02508_amd import binding

NUM_CLASSES, FREQ_DIM, LATENT_C, PATCH = 1000, 256, 4, 2
# (hidden, heads) of the transformer widths that are run; the MLP is four times as wide
SMALL, MEDIUM, LARGE = (384, 6), (768, 12), (1152, 16)


def _net(width, depth, h, w, bits=8):
    return {"hidden": width[0], "heads": width[1], "depth": depth, "latent_h": h, "latent_w": w, "bits": bits}


def _sample(name, net, latents, steps, interval, guidance=0.0, cache="fp32", stream="fp32", kind="sample"):
    c = {"kind": kind, "latents": latents, "steps": steps, "interval": interval, "guidance": guidance, "cache": cache,
         "stream": stream, **net}
    return {"name": name, **c} if name else c


def listed():
    xl = _net(LARGE, 28, 32, 32)
    return [
        # one small block, one latent, a refresh and a cached step: the latency of a call that has almost no work
        _sample("small block, 1 latent", _net(SMALL, 1, 32, 32), 1, 2, 2, kind="steps"),
        # a layer called by itself on a ragged batch of rows, packed 4-bit weights
        {"name": "linear 4-bit, 333 rows", "kind": "linear", "M": 333, "N": 1160, "K": 1168, "bits": 4},
        # the same at the size of a large batch's MLP: 64 latents of 256 tokens
        {"name": "linear 8-bit, 16384 rows", "kind": "linear", "M": 16384, "N": 4608, "K": 1152, "bits": 8},
        # one image, interactively: 50 steps, cache refreshed every 2nd
        _sample("sample 256, 1 latent", xl, 1, 50, 2),
        # the benchmark's run: 8 images at 256 pixels, 50 steps, cache refreshed every 2nd
        _sample("sample 256, 8 latents", xl, 8, 50, 2),
        # throughput with classifier-free guidance (128 rows of 256 tokens), refreshed every 3rd step; a real run has 100
        # steps, which only repeat these
        _sample("sample 256, 64 guided", xl, 64, 9, 3, guidance=1.5),
        # 512 pixels, 1024 tokens: attention counts; a real run has 50 steps
        _sample("sample 512, 16 latents", _net(LARGE, 28, 64, 64), 16, 10, 2),
        # 4-bit weights, refreshed every 5th step; a real run has 250 steps
        _sample("sample 256 4-bit, 32 latents", _net(LARGE, 28, 32, 32, 4), 32, 20, 5),
        # not square, a token count that no tile divides, guidance, bfloat16 cache and residual stream
        _sample("sample 400x272 bf16, 5 guided", _net(LARGE, 28, 50, 34), 5, 20, 2, guidance=4.0, cache="bf16", stream="bf16"),
        # the clustering of a small pool
        {"name": "cluster 1536", "kind": "cluster", "N": 1536, "F": 256, "n": 160, "m": 3, "k": 8},
        # and at the size the method is meant for: three subsamples of a twentieth, 100 clusters
        {"name": "cluster 32768", "kind": "cluster", "N": 32768, "F": 4096, "n": 1638, "m": 3, "k": 100},
        # set-up of a sampler: factors of the first steps of a schedule from two trajectories
        {"name": "fit 256, 2 latents", "kind": "fit", "latents": 2, "steps": 3, "interval": 2, "guidance": 0.0, **xl},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _rows(c):
    """Rows of the effective batch (guidance runs every latent twice)."""
    return c["latents"] * (2 if c["guidance"] > 0 else 1)


def _tokens(c):
    return (c["latent_h"] // PATCH) * (c["latent_w"] // PATCH)


def _n_full(c):
    return -(-c["steps"] // c["interval"])


def _block_flops(c):
    """Operations of one recomputed block: the five quantised linears and the attention."""
    D, rows, T = c["hidden"], _rows(c), _tokens(c)
    return 2.0 * rows * T * (4 * D * D + 8 * D * D) + 2.0 * rows * 6 * D * D + 4.0 * rows * T * T * D


def draw(rng):
    kind = rng.choice(("sample", "sample", "sample", "sample", "steps", "linear", "linear", "cluster", "fit"))
    if kind == "linear":
        M, N, K = _log_int(rng, 1, 32768), _log_int(rng, 16, 4608), 16 * _log_int(rng, 4, 288)
        while M * N * K > 16384 * 4608 * 1152:
            M = M * 3 // 4
        return {"kind": kind, "M": M, "N": N, "K": K, "bits": rng.choice((8, 8, 4))}
    if kind == "cluster":
        N, F, k = _log_int(rng, 1200, 32768), 4 * _log_int(rng, 16, 1024), _log_int(rng, 4, 100)
        return {"kind": kind, "N": N, "F": F, "n": max(N // 20, _tap_block(k), 128) | rng.randint(0, 1), "m": 3, "k": k}
    width = rng.choice((SMALL, MEDIUM, LARGE, LARGE))
    if kind == "steps":
        return _sample(None, _net(width, rng.randint(1, 4), 2 * rng.randint(4, 32), 2 * rng.randint(4, 32)), _log_int(rng, 1, 8),
                       rng.randint(2, 6), rng.randint(1, 3), rng.choice((0.0, 1.5)), kind=kind)
    net = _net(width, _log_int(rng, 6, 28), 2 * rng.randint(8, 32), 2 * rng.randint(8, 32), rng.choice((8, 8, 4)))
    if kind == "fit":
        c = {"kind": kind, "latents": rng.randint(1, 3), "steps": rng.randint(2, 4), "interval": 2, "guidance": 0.0, **net}
        while c["latents"] * c["steps"] * _tokens(c) > 2 * 3 * 256:
            c["latent_h"] -= 2 * (c["latent_h"] > 8)
            c["latent_w"] -= 2 * (c["latent_w"] > 8)
        return c
    fmt = rng.choice(("fp32", "fp32", "bf16"))
    c = _sample(None, net, _log_int(rng, 1, 64), _log_int(rng, 4, 50), rng.randint(1, 5), rng.choice((0.0, 1.5, 4.0)), fmt, fmt)
    c["latents"] = max(1, min(c["latents"], 32768 // (_tokens(c) * (2 if c["guidance"] > 0 else 1))))
    most = next(x for x in listed() if x["name"] == "sample 256, 64 guided")
    while c["steps"] > 1 and _n_full(c) * c["depth"] * _block_flops(c) > 0.9 * _n_full(most) * most["depth"] * _block_flops(most):
        c["steps"] -= 1
    return c


# ------------------------------------------------------------------------------------------------ preparation
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _randn(g, *shape, std=1.0):
    return torch.randn(shape, generator=g, device="cuda") * std


def _positions(h, w, D):
    """The fixed two-dimensional sine / cosine position table [h * w, D]."""
    q = D // 4
    omega = 10000.0 ** (-torch.arange(q, dtype=torch.float64) / q)
    y, x = torch.meshgrid(torch.arange(h, dtype=torch.float64), torch.arange(w, dtype=torch.float64), indexing="ij")
    parts = [f(p.reshape(-1, 1) * omega) for p in (x, y) for f in (torch.sin, torch.cos)]
    out = torch.zeros(h * w, D)
    out[:, :4 * q] = torch.cat(parts, 1).float()
    return out.cuda()


def _weights(m, g):
    """Random network parameters on the GPU, as the C interface takes them; the tensors to keep alive come second."""
    D, R, std = m.hidden, m.mlp_dim, 0.02
    n_out = m.patch * m.patch * 2 * m.latent_c
    dev = {"pos": _positions(m.latent_h // m.patch, m.latent_w // m.patch, D)}
    for k, s in {"patch_w": (D, m.latent_c * m.patch ** 2), "patch_b": (D,), "t_w1": (D, m.freq_dim), "t_b1": (D,), "t_w2": (D, D),
                 "t_b2": (D,), "label_table": (m.num_classes + 1, D), "fada_w": (2 * D, D), "fada_b": (2 * D,), "flin_w": (n_out, D),
                 "flin_b": (n_out,)}.items():
        dev[k] = _randn(g, *s, std=std)
    shapes = {"ada": (6 * D, D), "qkv": (3 * D, D), "proj": (D, D), "fc1": (R, D), "fc2": (D, R)}
    blocks = []
    for _ in range(m.depth):
        b = {}
        for k, (n, kk) in shapes.items():
            b[k + "_w"], b[k + "_b"] = _randn(g, n, kk, std=std), _randn(g, n, std=std)
        blocks.append(b)
    arr = (binding.BlockWeights * m.depth)()
    for i, b in enumerate(blocks):
        for k, t in b.items():
            setattr(arr[i], k, t.data_ptr())
    ws = binding.Weights()
    for k, t in dev.items():
        setattr(ws, k, t.data_ptr())
    ws.blocks = ctypes.cast(arr, ctypes.POINTER(binding.BlockWeights))
    return ws, (dev, blocks, arr)


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def _ok(rc):
    if rc:
        raise qc.QCError(rc, qc.last_error())


def _sampler(case, g):
    """A loaded and calibrated context, and the float32 weights."""
    m = SimpleNamespace(depth=case["depth"], hidden=case["hidden"], heads=case["heads"], mlp_dim=4 * case["hidden"], patch=PATCH,
                        latent_c=LATENT_C, latent_h=case["latent_h"], latent_w=case["latent_w"], num_classes=NUM_CLASSES,
                        freq_dim=FREQ_DIM, weight_bits=case["bits"], tokens=_tokens(case))
    ctx = qc.Context(m, _rows(case), case["interval"])
    ws, keep = _weights(m, g)
    _ok(qc.lib.qc_load_weights_f32(ctx.h, ctypes.byref(ws), _stream()))
    n = 2
    x = _randn(g, n, LATENT_C, m.latent_h, m.latent_w)
    t, y = (ctypes.c_int32 * n)(*[980 - 960 * i // (n - 1) for i in range(n)]), (ctypes.c_int32 * n)(*[7 + 500 * i for i in range(n)])
    _ok(qc.lib.qc_calibrate_minmax(ctx.h, ctypes.byref(ws), ctypes.c_void_p(x.data_ptr()), t, y, n, _stream()))
    return ctx, ws, keep


def _tap_block(k):
    """Iteration block of the clustering: k rounded up to a multiple of 8 plus 24 guard vectors, at most 128."""
    return min(128, (k + 7) // 8 * 8 + 24)


def _pool(case, g):
    """Intermediate samples of a diffusion sampler: the signal of a sample's class fades into noise as its time grows.  The
    pool covers somewhat fewer classes than there are clusters (the others go to time)."""
    N, F, k = case["N"], case["F"], case["k"]
    classes = max(2, k * 4 // 5)
    proto = _randn(g, classes, F)
    cls = torch.randperm(N, generator=g, device="cuda") % classes
    t = torch.randint(0, 50, (N,), generator=g, device="cuda") / 50.0
    a = torch.cos(0.5 * math.pi * (t + 0.01)).square()[:, None]
    X = a.sqrt() * proto[cls] + (1 - a).sqrt() * _randn(g, N, F)
    return X.contiguous(), t.float().contiguous()


def prepare(case, seed):
    g = _gen(seed)
    s = {"case": case}
    kind = case["kind"]
    if kind == "linear":
        M, N, K, bits = case["M"], case["N"], case["K"], case["bits"]
        s.update(x=_randn(g, M, K), q=torch.empty((M, K), dtype=torch.int8, device="cuda"), y=torch.empty((M, N), device="cuda"),
                 bias=_randn(g, N, std=0.02), scale=0.04, zp=121, wscale=torch.empty(N, device="cuda"),
                 qw=torch.empty((N, K * bits // 8), dtype=torch.int8, device="cuda"),
                 wsum=torch.empty(N, dtype=torch.int32, device="cuda"))
        qc.qc_quantize_weight(_randn(g, N, K, std=0.02), bits, s["qw"], s["wscale"], s["wsum"])
        return s
    if kind == "cluster":
        N, n, m, k = case["N"], case["n"], case["m"], case["k"]
        kb = _tap_block(k)
        X, t = _pool(case, g)
        pick = lambda count: torch.stack([torch.randperm(N, generator=g, device="cuda")[:count] for _ in range(m)])  # noqa: E731
        slots = min(m, 3)
        room = (qc.qc_tap_workspace_bytes(N, case["F"], n, k, kb) + 255) // 256 * 256
        s.update(X=X, t=t, subs=pick(n).sort(dim=1).values.int().contiguous(), init=pick(k).int().contiguous(), q0=_randn(g, kb, n),
                 work=torch.empty(slots * room, dtype=torch.uint8, device="cuda"), labels=torch.empty(N, dtype=torch.int32, device="cuda"),
                 per=torch.empty((m, N), dtype=torch.int32, device="cuda"))
        return s
    s["ctx"], ws, keep = _sampler(case, g)
    B = case["latents"]
    s["x"] = _randn(g, B, LATENT_C, case["latent_h"], case["latent_w"])
    s["labels"] = torch.randint(0, NUM_CLASSES, (B,), generator=g, device="cuda", dtype=torch.int32)
    s["K"] = 0.95 + 0.05 * torch.rand((case["steps"], LATENT_C), generator=g, device="cuda")
    if kind == "fit":
        s.update(ws=ws, keep=keep)
    else:
        torch.cuda.synchronize()                # the float32 weights are given back
        s["ctx"].set_cache_format(case["cache"])
        s["ctx"].set_stream_format(case["stream"])
        s["schedule"] = list(zip(*qc.qc_ddim_schedule(case["steps"])))
    return s


# ------------------------------------------------------------------------------------------------------- a pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "linear":
        qc.qc_quantize_act(s["x"], s["q"], s["scale"], s["zp"])
        qc.qc_w8a8_linear(s["q"], s["qw"], s["wsum"], s["wscale"], s["bias"], s["scale"], s["zp"], case["bits"], s["y"])
        return s["q"], s["y"]
    if kind == "cluster":
        qc.qc_tap_cluster(s["X"], s["t"], s["subs"], 0.5, case["k"], 8, s["q0"], s["init"], 100, s["labels"], s["per"], s["work"])
        return s["labels"], s["per"]
    x = s["x"].clone()
    if kind == "sample":
        s["ctx"].sample(x, s["labels"], case["steps"], case["guidance"], s["K"])
        return x
    if kind == "steps":
        for i, (t, at, ap) in enumerate(s["schedule"]):
            s["ctx"].sample_step(x, s["labels"], i, t, at, ap, case["guidance"], s["K"][i])
        return x
    ref, K = s["x"].clone(), torch.empty_like(s["K"])
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    _ok(qc.lib.qc_vc_fit_sampler(s["ctx"].h, ctypes.byref(s["ws"]), ptr(x), ptr(ref), ptr(s["labels"]), x.shape[0], case["steps"],
                                 case["guidance"], 1e-3, ptr(K), _stream()))
    return x, ref, K


# ------------------------------------------------------------------------------------------- what a pass needs
def work(case):
    kind = case["kind"]
    if kind == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 5.0 * M * K + N * K * case["bits"] / 8 + 12.0 * N + 4.0 * M * N, "flops": 2.0 * M * N * K}
    if kind == "cluster":
        # similarity, L^T L (one triangle), block power iteration, projection; k-means is small beside them
        N, F, n, m, k = (case[v] for v in ("N", "F", "n", "m", "k"))
        kb = _tap_block(k)
        return {"bytes": 4.0 * N * F + 4.0 * m * n + 4.0 * (m + 1) * N,
                "flops": m * (2.0 * N * n * F + 1.0 * n * n * N + 8 * 2.0 * kb * n * n + 2.0 * N * n * k)}
    D, L, T, rows = case["hidden"], case["depth"], _tokens(case), _rows(case)
    n_full, M = _n_full(case), _rows(case) * _tokens(case)
    n_cached = case["steps"] - n_full
    wb = case["bits"] / 8
    lat = 4.0 * LATENT_C * case["latent_h"] * case["latent_w"]
    module = 2.0 * M * D * (2 if case.get("cache") == "bf16" else 4)      # both stored module outputs of a block
    # the block weights once per refresh step (they exceed every cache of the chip), the adaLN weights once for all steps;
    # the stored outputs are written by a refresh step that is followed by a reuse and read once per cached step
    data = L * (n_full * 12 * D * D * wb + 6 * D * D * wb + (min(n_full, n_cached) + n_cached) * module) + 2.0 * case["latents"] * lat
    ops = L * (n_full * _block_flops(case) + n_cached * (2.0 * rows * 2 * D * D + 4.0 * M * D))
    if kind == "fit":
        data += case["steps"] * L * 4.0 * 18 * D * D + 2.0 * case["latents"] * lat
        ops += case["steps"] * L * _block_flops(case)
    return {"bytes": data, "flops": ops}


def tolerance(case):
    kind = case["kind"]
    if kind == "linear":        # codes and integer sums are exact; the float32 results round once
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    if kind == "cluster":       # labels: a sample at equal distance from two centres may go either way, and moves its centres
        return {"rel": 0.0, "differ": 0.01}
    if kind == "fit":           # the trajectories part where the float32 factors move an 8-bit code
        return {"rel": 3e-3, "max": 3e-2}
    return {"rel": 1e-3, "max": 2e-2}       # 8-bit codes: one that differs moves a latent by about 1e-3
