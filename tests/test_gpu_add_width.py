"""GPU parity of the adding passes that count symbols in both their widths (512 and 256 threads a workgroup), against the CPU
oracle: messages on both sides of the switch, frames of whole blocks, ragged and odd frames, many small ones; two and
three streams, the ring step plain, stochastic and with the predictor; frames of every codec, frequent escapes, sums past 16 bits
and past 2^30, RAW operands, local values that cannot be quantized."""
import numpy as np
import pytest

import oracle
from paper_2605_12396_amd import workloads as W
from test_gpu_escape_sums import _message as _escapes
from test_gpu_reduce_k import check
from test_gpu_sr import _gpu_reduce_local_sr

pytestmark = pytest.mark.gpu

# (elements, frame length): 256 threads; and the neighbours that take 512
SMALL = [(917505, 262144), (1048576 + 2050, 262144), (1 << 20, 1 << 20), (983040 + 300, 65536), (1000003, 100003), (920001, 1500)]
LARGE = [(917504, 262144), (1000003, 16384), (921600, 70000)]
KINDS = ["huffman", "escapes", "all escapes", "fixed", "wide", "raw", "delta", "delta fixed", "alphabet 1024"]


@pytest.fixture(scope="module")
def nz(gpu_device):
    from paper_2605_12396_amd import binding
    binding.lib()
    return binding


def _operands(kind, n, eb, kw):
    """Two streams and the local message of a ring step."""
    o = oracle.make_opts(**kw)
    forced = lambda c: oracle.make_opts(force_codec=c, **kw)  # noqa: E731
    if kind in ("fixed", "delta fixed", "wide"):
        xs = [(6.0 if kind == "wide" else 1.0) * W.sweep_payload("uniform", n, 31 + p) for p in range(3)]
        ss = [oracle.compress(x.astype(np.float32), eb, forced(1))[0] for x in xs]
        if kind == "wide":       # codes of 17 bits in a FIXEDLEN frame, sums past 16 bits
            ss[0] = oracle.reduce_k([ss[0], ss[2]], n, eb, forced(1))[0]
    elif kind in ("escapes", "all escapes"):
        xs = [_escapes(n, 0.08 if kind == "escapes" else 1.0, 60 + p) for p in range(3)]
        ss = [oracle.compress(x, eb, forced(2))[0] for x in xs]
    else:
        xs = [W.gradient_like(n, seed=70 + p) for p in range(3)]
        if kind == "raw":        # the first frame, one in the middle and the last one, in either operand
            xs[0][[3, n - 1]] = np.nan, np.inf
            xs[1][[n // 2, n - 1]] = np.nan, -np.inf
        ss = [oracle.compress(x, eb, o)[0] for x in xs]
    return ss[:2], xs[2].astype(np.float32)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n,chunk", SMALL + LARGE)
def test_parity(nz, n, chunk, kind):
    import torch
    eb = 1e-4
    kw = dict(chunk_elems=chunk)
    if kind.startswith("delta"):
        kw["predictor"] = 1
    if kind == "alphabet 1024":
        kw["alphabet"] = 1024
    g, o = nz.make_opts(**kw), oracle.make_opts(**kw)
    ss, x = _operands(kind, n, eb, kw)
    check(nz, ss, n, eb, **kw)
    check(nz, [ss[1], ss[1], ss[0]], n, eb, **kw)
    ds = torch.from_numpy(np.concatenate([ss[0], np.zeros((-ss[0].size) % 16, np.uint8)])).to("cuda:0")
    sess = nz.Session(n, g, "cuda:0", reduce=True)
    for bad in (False, True):
        if bad:                  # frames whose local data cannot be quantized
            x = x.copy()
            x[[n // 3, n - 2]] = np.nan, 1e9
        ref, ores, orc = oracle.reduce_local(ss[0], x, eb, o)
        rc, out = sess.reduce_local(ds, ss[0].size, torch.from_numpy(x).to("cuda:0"), n, eb)
        r = sess.result()
        assert rc == 0 and orc == 0 and r["status"] == 0 and r["bytes"] == ores.bytes
        assert (r["n_raw"], r["n_fixed"], r["n_huff"]) == (ores.n_raw, ores.n_fixed, ores.n_huff)
        assert np.array_equal(out[:r["bytes"]].cpu().numpy(), ref)
        if not kind.startswith("delta"):
            step = oracle.step_constants(eb)[0]
            ref, ores, orc = oracle.reduce_local_sr(ss[0], x, step, 8, o)
            rc, r, got = _gpu_reduce_local_sr(nz, ss[0], x, float(step), 8, g)
            assert rc == 0 and orc == 0 and r["status"] == 0 and r["bytes"] == ores.bytes
            assert np.array_equal(got, ref)


@pytest.mark.parametrize("n,chunk", [SMALL[1], LARGE[1]])
def test_sums_past_the_range(nz, n, chunk):
    """Codes of 2^29 doubled twice: the last operand's pass finds the sum out of range and the frame turns RAW."""
    eb, kw = 1e-3, dict(chunk_elems=chunk)
    o = oracle.make_opts(**kw)
    step, _ = oracle.step_constants(eb)
    y = np.zeros(n, np.float32)
    y[[3, 4, 70000, n - 1]] = step, -step, step, step
    t = oracle.compress(y, eb, o)[0]
    for _ in range(29):
        t = oracle.reduce_frames(t, t, n, eb, o)[0]
    check(nz, [t, t], n, eb, **kw)                                       # 2^30 exactly: still a code
    ref, ores = check(nz, [t, t, t], n, eb, **kw)
    assert ores.n_raw >= 2
