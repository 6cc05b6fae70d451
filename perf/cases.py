"""What the compression path is measured on: messages a rank hands to its collectives, through the public entry points.

A rank of a compressed collective does four things with a message: it compresses its own data (nz_compress, or the sampled
nz_compress_rea, or the stochastic nz_compress_sr), folds incoming streams into it (nz_reduce_local in a ring,
nz_reduce_frames and nz_reduce_k where several streams meet), and decompresses the result (nz_decompress).  The cases are
these calls on the payloads of paper_2605_12396_amd/workloads.py, drawn on the GPU, from the smallest message of the size
sweep (64 KB) to a 512 MB field.  Messages are plain float32; every result is bytes or a single float32 product, so
all outputs are exact.
"""
import math

import torch

from paper_2605_12396_amd import binding as nz

SMALLEST = 16 << 10              # elements: the 64 KB message of the size sweep
LARGEST = 64 << 20               # elements of a drawn message: the 256 MB gradient
CALIBRATION = 65536              # elements of the message that the sampled path's Huffman context is built from

# (op, weight in draw)
OPS = (("compress", 4), ("decompress", 4), ("roundtrip", 2), ("reduce_local", 3), ("reduce_frames", 2), ("reduce_k", 2),
       ("compress_rea", 2), ("reduce_local_rea", 1), ("qsgd", 2))


def _case(name, op, n, data, bound, rel=False, chunk=0, alphabet=0, predictor=0, k=2):
    """bound: absolute error bound, or relative to the message's range (rel), or levels per sign of the norm (qsgd);
    chunk: elements per frame (0: the default, 1 MiB); alphabet: Huffman alphabet (0: the default, 256)."""
    c = {"op": op, "n": n, "data": data, "bound": bound, "rel": rel, "chunk": chunk, "alphabet": alphabet, "predictor": predictor,
         "k": k}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest message of the size sweep, one frame: nothing but latency
        _case("compress-64KB", "compress", 16384, "laplace", 1e-4),
        # a small field in 64 KiB frames that stay fixed-length, there and back
        _case("field-4MB-roundtrip", "roundtrip", 256 * 64 * 64, "field", 1e-4, chunk=16384),
        # a bucket of gradients in a ring, a few frames and a ragged end
        _case("ring-step-1MB-sampled", "reduce_local_rea", 300007, "laplace", 1e-4),
        # a line of a smooth signal with the delta predictor, there and back
        _case("line-4MB-delta-roundtrip", "roundtrip", 1 << 20, "sinusoid", 1e-4, predictor=1),
        # stochastic quantizer: width from the norm, read back by the host (ranks agree on it), then the stream
        _case("qsgd-10MB", "qsgd", 2500001, "laplace", 1024),
        # ring step on a bucket of gradients with outliers, odd size
        _case("ring-step-44MB", "reduce_local", 11000003, "gradient", 1e-4, rel=True),
        # the sampled arbitration on a 64 MB message
        _case("compress-64MB-sampled", "compress_rea", (16 << 20) + 77, "gradient", 1e-4, rel=True),
        # two incoming streams folded, about ten bits a symbol
        _case("reduce-2x128MB", "reduce_frames", 32 << 20, "laplace", 1e-5),
        # eight peers' chunks folded at once, as a direct reduce-scatter delivers them
        _case("reduce-8x128MB", "reduce_k", 32 << 20, "laplace", 1e-5, k=8),
        # the 256 MB gradient, sender and receiver
        _case("compress-256MB", "compress", 64 << 20, "gradient", 1e-4, rel=True),
        _case("decompress-256MB", "decompress", 64 << 20, "gradient", 1e-4, rel=True),
        # a 512^3 field at a tight relative bound, there and back: the largest
        _case("field-512MB-roundtrip", "roundtrip", 512 ** 3, "grf", 1e-3, rel=True),
    ]


def draw(rng):
    op = rng.choices([o for o, _ in OPS], [w for _, w in OPS])[0]
    top = LARGEST // 4 if op == "reduce_k" else LARGEST
    n = int(round(math.exp(rng.uniform(math.log(SMALLEST), math.log(top)))))
    if rng.random() < 0.4:
        n = max(SMALLEST, n // 4096 * 4096)                    # tensors padded to a round size, as buckets are
    n = min(n, top)
    if op == "qsgd":
        return _case(None, op, n, rng.choice(("laplace", "gradient")), rng.choice((256, 1024, 4096)))
    data = rng.choice(("laplace", "laplace", "gradient", "gradient", "uniform", "sinusoid", "field", "grf"))
    predictor = 0
    if data in ("field", "grf"):
        n = max(26, min(400, int(round(n ** (1 / 3))))) ** 3   # cubes
    if data == "sinusoid" and not op.endswith("_rea") and rng.random() < 0.5:
        predictor = 1
    rel = data in ("gradient", "grf")
    bound = {"laplace": (1e-5, 1e-4), "gradient": (1e-4,), "uniform": (1e-4, 1e-3), "sinusoid": (1e-4,), "field": (1e-4, 1e-3),
             "grf": (1e-2, 1e-3, 1e-4)}[data]
    chunk = rng.choices((0, 16384, 1 << 20), (4, 2, 1))[0]     # 1 MiB frames, 64 KiB frames, the 4 MiB channel buffer
    alphabet = rng.choices((0, 1024), (5, 1))[0]
    return _case(None, op, n, data, rng.choice(bound), rel, chunk, alphabet, predictor, rng.choice((3, 4, 8)) if op == "reduce_k" else 2)


# ---- messages ----

def _laplace(gen, n, b, device):
    u = torch.rand(n, generator=gen, device=device) - 0.5
    return u.sign() * torch.log1p(-2.0 * u.abs().clamp(max=0.5 - 2.0 ** -25)) * -b


def _waves(gen, axes, device):
    """Sum of four plane waves of random phase, whole wavenumbers 1..8 along each axis, and noise of 1e-3."""
    out = None
    for _ in range(4):
        k = torch.randint(1, 9, (len(axes),), generator=gen, device=device)
        arg = torch.rand(1, generator=gen, device=device)
        for i, a in enumerate(axes):
            arg = arg + k[i] * a
        out = torch.sin(2.0 * math.pi * arg) if out is None else out + torch.sin(2.0 * math.pi * arg)
    return (out + 1e-3 * torch.randn(out.shape, generator=gen, device=device)).reshape(-1)


def _message(data, n, seed, device="cuda", count=None):
    """The message of `n` elements, or its first `count`."""
    gen = torch.Generator(device=device)
    gen.manual_seed(seed)
    m = n if count is None else min(n, count)
    if data == "laplace":                                      # gradients
        x = _laplace(gen, m, 1e-3, device)
    elif data == "gradient":                                   # gradients with 1 % of outliers a hundred times as large
        x = _laplace(gen, m, 1e-3, device)
        out = torch.rand(m, generator=gen, device=device) < 0.01
        x = torch.where(out, _laplace(gen, m, 1e-1, device), x)
    elif data == "uniform":
        x = torch.rand(m, generator=gen, device=device) * 2.0 - 1.0
    elif data == "sinusoid":
        x = _waves(gen, [torch.arange(m, device=device, dtype=torch.float64) / n], device)
    elif data == "field":
        side = round(n ** (1 / 3))
        shape = (side, side, side) if side ** 3 == n else (n // 4096, 64, 64)
        shape = shape if count is None else (max(1, m // (shape[1] * shape[2])), shape[1], shape[2])
        full = (side, side, side) if side ** 3 == n else (n // 4096, 64, 64)
        axes = [(torch.arange(s, device=device, dtype=torch.float32) / f).view([-1 if i == a else 1 for i in range(3)])
                for a, (s, f) in enumerate(zip(shape, full))]
        x = _waves(gen, axes, device)
    elif count is not None:                                    # one-point distribution of the random field
        x = torch.randn(m, generator=gen, device=device)
    else:                                                      # Gaussian random field, P(k) ~ k^-3, unit variance
        side = round(n ** (1 / 3))
        f = torch.fft.rfftn(torch.randn((side, side, side), generator=gen, device=device))
        k = torch.fft.fftfreq(side, 1.0 / side, device=device)
        k2 = k[:, None, None] ** 2 + k[None, :, None] ** 2 + torch.fft.rfftfreq(side, 1.0 / side, device=device)[None, None, :] ** 2
        k2[0, 0, 0] = 1.0
        amp = k2 ** -0.75
        amp[0, 0, 0] = 0.0
        x = torch.fft.irfftn(f * amp, s=(side, side, side)).reshape(-1)
        x = (x - x.mean()) / x.std()
    return x.to(torch.float32).contiguous()


# ---- states and passes ----

def prepare(case, seed):
    op, n, k = case["op"], case["n"], case["k"]
    opts = nz.make_opts(chunk_elems=case["chunk"], alphabet=case["alphabet"], predictor=case["predictor"])
    rea = op.endswith("_rea")
    xs = [_message(case["data"], n, seed * 64 + p) for p in range({"reduce_k": k, "reduce_frames": 2, "reduce_local": 2,
                                                                   "reduce_local_rea": 2}.get(op, 1))]
    n = xs[0].numel()
    eb = float(case["bound"])
    if case["rel"]:
        eb *= float(xs[0].max() - xs[0].min())
    bytes_of = lambda b: torch.zeros(b, dtype=torch.uint8, device="cuda")  # noqa: E731
    s = {"op": op, "n": n, "opts": opts, "eb": eb, "seed": seed & 0x7FFFFFFF, "cap": nz.nz_compress_bound(n, opts),
         "res": bytes_of(max(nz.RESULT_BYTES, nz.REA_RESULT_BYTES))}
    need = max(nz.nz_reduce_workspace_bytes(n, opts) if op.startswith("reduce") else nz.nz_workspace_bytes(n, opts), 8192)
    if rea:
        need = max(need, nz.nz_rea_workspace_bytes(n, opts), nz.nz_reduce_rea_workspace_bytes(n, opts) if op == "reduce_local_rea" else 0)
        s["ctx"] = bytes_of(nz.nz_context_bytes())
    s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    s["ws_bytes"] = need
    if op != "decompress":
        s["out"] = bytes_of(s["cap"])
    if op in ("decompress", "roundtrip"):
        s["y"] = torch.zeros(n, dtype=torch.float32, device="cuda")
        s["yres"] = bytes_of(nz.RESULT_BYTES)
    if op == "qsgd":
        s["levels"] = int(case["bound"])
        s["step"] = torch.zeros(1, dtype=torch.float32, device="cuda")
    if rea:       # the communicator's cached context: the code of a calibration message, here what arrives first
        m = min(n, CALIBRATION)
        sample = xs[0][:m] + xs[1][:m] if op == "reduce_local_rea" else xs[0][:m]
        if nz.nz_context_build(sample, m, eb, opts, s["ctx"], s["ws"], need):
            raise RuntimeError("nz_context_build failed")
    if op in ("decompress", "reduce_frames", "reduce_k", "reduce_local", "reduce_local_rea"):
        incoming = xs if op in ("decompress", "reduce_frames", "reduce_k") else xs[:1]
        buf, s["streams"], s["sizes"] = bytes_of(s["cap"]), [], []
        for x in incoming:                                     # what the peers send
            rc = nz.nz_compress(x, n, eb, buf, s["cap"], s["res"], opts, s["ws"], need)
            r = nz.read_result(s["res"])
            if rc or r["status"]:
                raise RuntimeError("nz_compress failed: %s %s" % (rc, r))
            s["streams"].append(buf[:r["bytes"]].clone())
            s["sizes"].append(r["bytes"])
        s["res"].zero_()
    if op in ("compress", "roundtrip", "compress_rea", "qsgd"):
        s["x"] = xs[0]
    if op.startswith("reduce_local"):
        s["x"] = xs[1]
    return s


def _checked(rc):
    if rc:
        raise RuntimeError("the call was refused: %d" % rc)


def run(state):
    s = state
    op, n, eb, opts, ws, wsb = s["op"], s["n"], s["eb"], s["opts"], s["ws"], s["ws_bytes"]
    if op == "compress":
        _checked(nz.nz_compress(s["x"], n, eb, s["out"], s["cap"], s["res"], opts, ws, wsb))
    elif op == "decompress":
        _checked(nz.nz_decompress(s["streams"][0], s["sizes"][0], s["y"], n, eb, s["yres"], opts, ws, wsb))
        return {"y": s["y"], "res": s["yres"]}
    elif op == "roundtrip":                                    # (the stream's own header says where it ends)
        _checked(nz.nz_compress(s["x"], n, eb, s["out"], s["cap"], s["res"], opts, ws, wsb))
        _checked(nz.nz_decompress(s["out"], s["cap"], s["y"], n, eb, s["yres"], opts, ws, wsb))
        return {"stream": s["out"], "res": s["res"], "y": s["y"], "yres": s["yres"]}
    elif op == "reduce_frames":
        _checked(nz.nz_reduce_frames(s["streams"][0], s["sizes"][0], s["streams"][1], s["sizes"][1], s["out"], s["cap"], n, eb,
                                     s["res"], opts, ws, wsb))
    elif op == "reduce_k":
        _checked(nz.nz_reduce_k(s["streams"], s["sizes"], s["out"], s["cap"], n, eb, s["res"], opts, ws, wsb))
    elif op == "reduce_local":
        _checked(nz.nz_reduce_local(s["streams"][0], s["sizes"][0], s["x"], s["out"], s["cap"], n, eb, s["res"], opts, ws, wsb))
    elif op == "compress_rea":
        _checked(nz.nz_compress_rea(s["x"], n, eb, s["ctx"], s["out"], s["cap"], s["res"], opts, None, ws, wsb))
    elif op == "reduce_local_rea":
        _checked(nz.nz_reduce_local_rea(s["streams"][0], s["sizes"][0], s["x"], n, eb, s["ctx"], s["out"], s["cap"], s["res"],
                                        opts, None, ws, wsb))
    else:                                                      # qsgd: the width is a host number of the next call
        _checked(nz.nz_qsgd_step(s["x"], n, s["levels"], s["step"], ws, wsb))
        step = s["step"].item()
        _checked(nz.nz_compress_sr(s["x"], n, step, s["seed"], s["out"], s["cap"], s["res"], opts, ws, wsb))
        return {"stream": s["out"], "res": s["res"], "step": s["step"]}
    return {"stream": s["out"], "res": s["res"]}


# ---- what a pass cannot do without ----

def _stream_bytes(case, operands):
    """Size of the stream of a sum of `operands` messages, from the code statistics of 64 Ki elements of such messages."""
    n, K = case["n"], case["alphabet"] or 256
    total = None
    for p in range(operands):
        x = _message(case["data"], n, 1 + p, device="cpu", count=65536)
        eb = float(case["bound"])
        if case["op"] == "qsgd":
            step = float(x.double().square().mean().sqrt()) * math.sqrt(n) / eb
        else:
            if case["rel"]:      # extremes of n values: the outliers' Laplace tails, or a field's few large modes
                eb *= 0.2 * math.log(max(2.0, 0.01 * n)) if case["data"] == "gradient" else 8.0
            step = eb * 63 / 32
        q = torch.round(x / step).to(torch.int64)
        if case["predictor"]:
            q[1:] = q[1:] - q[:-1]
        total = q if total is None else total + q
    z = torch.where(total >= 0, 2 * total, -2 * total - 1)
    counts = torch.bincount(z.clamp(max=K - 1), minlength=K).double()
    p = counts[counts > 0] / counts.sum()
    bits = float(-(p * p.log2()).sum()) + 32.0 * float(counts[K - 1] / counts.sum()) + 1.0 / 16
    bits = min(bits, 32.0, math.ceil(math.log2(int(z.max()) + 1)) if int(z.max()) else 0.0) if bits > 8 else max(bits, 1.0)
    return n * bits / 8.0 + 200.0


def work(case):
    op, n = case["op"], case["n"]
    s1 = _stream_bytes(case, 1)
    if op in ("compress", "decompress", "compress_rea", "qsgd"):
        b = 4.0 * n + s1
    elif op == "roundtrip":
        b = 8.0 * n + 2.0 * s1
    elif op.startswith("reduce_local"):
        b = s1 + 4.0 * n + _stream_bytes(case, 2)
    else:
        b = case["k"] * s1 + _stream_bytes(case, case["k"])
    return {"bytes": b, "flops": 0.0}


def tolerance(case):
    return "exact"
