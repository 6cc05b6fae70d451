"""GPU parity of RAW frames taken four elements at a time, against the CPU oracle: decompression and every pass of the reduces, RAW as
the first, a middle or the last operand beside HUFFMAN and FIXEDLEN frames (codes past 16 bits among them) and beside the rank's
own data, at the edges of what a thread has on its way at once and of a workgroup's block, and with frames that start off a
multiple of four.  NaN and infinities travel in RAW frames."""
import numpy as np
import pytest

import oracle
from paper_2605_12396_amd import workloads as W
from test_gpu_parity import gpu_decompress, gpu_reduce_local
from test_gpu_rea import check_ring_rea
from test_gpu_reduce_k import check
from test_gpu_sr import _gpu_reduce_local_sr

pytestmark = pytest.mark.gpu

# eight groups of 256 threads are 8192 elements, four groups of 512 as many: one short of a thread's last group, whole, one over
SHAPES = [(3, 0), (8192 - 3, 0), (8192, 0), (8192 + 1, 0), (8192 + 4096 - 1, 0), (65536 + 8192 - 1, 65536), (131072 + 8195, 262144),
          (262144 + 65537, 262144), (70001, 16384), (3 * 10003, 10003)]


@pytest.fixture(scope="module")
def nz(gpu_device):
    from paper_2605_12396_amd import binding
    binding.lib()
    return binding


def _special(x, seed):
    x = x.copy()
    rng = np.random.default_rng(seed)
    at = rng.integers(0, x.size, min(12, x.size))
    x[at] = rng.choice(np.array([np.nan, np.inf, -np.inf, -0.0, 1e30, -1e30, 1e-42], np.float32), at.size)
    return x


@pytest.mark.parametrize("n,chunk", SHAPES)
def test_decompress(nz, n, chunk):
    eb, o = 1e-4, oracle.make_opts(chunk_elems=chunk, force_codec=0)
    x = _special(W.sweep_payload("uniform", n, n % 89), n)
    s = oracle.compress(x, eb, o)[0]
    ref = oracle.decompress(s, n, eb)[0]
    rc, r, got = gpu_decompress(nz, s, n, eb, nz.make_opts(chunk_elems=chunk))
    assert rc == 0 and r["status"] == 0 and r["n_raw"] == r["n_frames"]
    assert (got.view(np.uint32) == ref.view(np.uint32)).all()


# what the other operands are coded as: HUFFMAN, FIXEDLEN, FIXEDLEN with codes that leave 16 bits once summed, RAW
@pytest.mark.parametrize("others", ["huffman", "fixed", "wide", "raw"])
@pytest.mark.parametrize("at", [0, 1, 2])
@pytest.mark.parametrize("n,chunk", SHAPES)
def test_reduce_k(nz, n, chunk, at, others):
    eb = 1e-4
    o = oracle.make_opts(chunk_elems=chunk, force_codec={"huffman": 2, "raw": 0}.get(others, 1))
    if others == "huffman":
        xs = [W.gradient_like(n, seed=50 + p) for p in range(3)]
    else:
        xs = [(W.sweep_payload("uniform", n, 60 + p) * (6.0 if others == "wide" else 1.0)).astype(np.float32) for p in range(3)]
    ss = [oracle.compress(x, eb, o)[0] for x in xs]
    ss[at] = oracle.compress(_special(xs[at], n + at), eb, oracle.make_opts(chunk_elems=chunk, force_codec=0))[0]
    check(nz, ss, n, eb, chunk_elems=chunk)
    check(nz, [ss[at], ss[(at + 1) % 3]] if at < 2 else [ss[0], ss[2]], n, eb, chunk_elems=chunk)


@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("n,chunk", SHAPES)
def test_ring_steps(nz, n, chunk, special):
    """The incoming frames RAW, the rank's own data quantized beside them, with and without values that cannot be."""
    eb, kw = 1e-4, dict(chunk_elems=chunk)
    a, x = W.sweep_payload("uniform", n, 5), W.gradient_like(n, seed=6)
    if special:
        a, x = _special(a, n), _special(x, n + 1)
    raw = dict(kw, force_codec=0)
    s = oracle.compress(a, eb, oracle.make_opts(**raw))[0]
    ref, ores, orc = oracle.reduce_local(s, x, eb, oracle.make_opts(**kw))
    rc, r, got = gpu_reduce_local(nz, s, x, eb, nz.make_opts(**kw))
    assert orc == 0 and rc == 0 and r["status"] == 0 and r["bytes"] == ores.bytes and (got == ref).all()
    check_ring_rea(nz, a, x, eb, a_kw=raw, **kw)
    step = float(np.float32(2e-4))
    ssr = oracle.compress_sr(a, step, 3, oracle.make_opts(**raw))[0]
    ref, ores, orc = oracle.reduce_local_sr(ssr, x, step, 4, oracle.make_opts(**kw))
    rc, r, got = _gpu_reduce_local_sr(nz, ssr, x, step, 4, nz.make_opts(**kw))
    assert orc == 0 and rc == 0 and r["status"] == 0 and r["bytes"] == ores.bytes and (got == ref).all()
