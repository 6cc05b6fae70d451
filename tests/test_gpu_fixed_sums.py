"""GPU parity of the reduces over FIXEDLEN frames, against the CPU oracle: every adding pass (staging, accumulating, last
operand, ring step plain / stochastic / sampled) at the edges of its passes, halves and blocks, with frames whose first
element is not a multiple of four, sums and operands past 16 bits, local values that cannot be quantized, alphabets that
the codes leave and alphabets that hold them, and the predictor."""
import numpy as np
import pytest

import oracle
from paper_2605_12396_amd import workloads as W
from test_gpu_rea import check_ring_rea
from test_gpu_reduce_k import check
from test_gpu_sr import _gpu_reduce_local_sr

pytestmark = pytest.mark.gpu

SHAPES = [(5, 0), (1023, 0), (2049, 0), (65535, 0), (65536, 65536), (65536 + 2047, 0), (131072, 0), (131072 + 2050, 262144),
          (262144 + 65537, 262144), (70001, 16384), (3 * 10003, 10003)]


@pytest.fixture(scope="module")
def nz(gpu_device):
    from paper_2605_12396_amd import binding
    binding.lib()
    return binding


def _messages(n, k, scale, seed):
    return [(scale * W.sweep_payload("uniform", n, seed + p)).astype(np.float32) for p in range(k)]


# scale 0.01: codes of at most 7 bits, inside the alphabet; 1: 14 bits, eight of them past 16; 6: 16 bits, two of them past 16
@pytest.mark.parametrize("scale,k,kw", [(0.01, 2, {}), (1.0, 2, {}), (1.0, 8, {}), (6.0, 3, dict(alphabet=1024)), (1.0, 3, dict(predictor=1))],
                         ids=["narrow", "two", "eight", "wide", "delta"])
@pytest.mark.parametrize("n,chunk", SHAPES)
def test_reduce_k(nz, n, chunk, scale, k, kw):
    eb, kw = 1e-4, dict(kw, chunk_elems=chunk)
    o = oracle.make_opts(force_codec=1, **kw)
    ss = [oracle.compress(x, eb, o)[0] for x in _messages(n, k, scale, 900 + n % 97)]
    ref, ores = check(nz, ss, n, eb, **kw)
    if scale == 6.0:       # the sum as an operand of its own: codes of 17 bits in a FIXEDLEN frame, in every place
        wide, _, rc = oracle.reduce_k(ss, n, eb, o)
        assert rc == 0
        for ops in ([wide, ss[0], ss[1]], [ss[0], wide, ss[1]], [ss[0], ss[1], wide], [wide, wide]):
            check(nz, ops, n, eb, **kw)


@pytest.mark.parametrize("bad", [False, True], ids=["", "unquantizable"])
@pytest.mark.parametrize("scale", [0.01, 6.0])
@pytest.mark.parametrize("n,chunk", SHAPES)
def test_ring_step(nz, n, chunk, scale, bad):
    eb, kw = 1e-4, dict(chunk_elems=chunk)
    g, o, of = nz.make_opts(**kw), oracle.make_opts(**kw), oracle.make_opts(force_codec=1, **kw)
    a, x = _messages(n, 2, scale, 950 + n % 89)
    if bad:
        x[n // 2] = np.nan
        x[n - 1] = 1e9
    s = oracle.compress(a, eb, of)[0]
    ref, ores, orc = oracle.reduce_local(s, x, eb, o)
    sess = nz.Session(n, g, "cuda:0", reduce=True)
    import torch
    ds = torch.from_numpy(np.concatenate([s, np.zeros((-s.size) % 16, np.uint8)])).to("cuda:0")
    rc, out = sess.reduce_local(ds, s.size, torch.from_numpy(x).to("cuda:0"), n, eb)
    r = sess.result()
    assert rc == 0 and orc == 0 and r["status"] == 0 and r["bytes"] == ores.bytes
    assert np.array_equal(out[:r["bytes"]].cpu().numpy(), ref)
    check_ring_rea(nz, a, x, eb, a_kw=dict(force_codec=1, **kw), **kw)
    step = float(np.float32(2e-4))
    ss, _, src = oracle.compress_sr(a, step, 7, of)
    ref, ores, orc = oracle.reduce_local_sr(ss, x, step, 8, o)
    rc, r, got = _gpu_reduce_local_sr(nz, ss, x, step, 8, g)
    assert src == 0 and rc == 0 and orc == 0 and r["status"] == 0 and r["bytes"] == ores.bytes
    assert np.array_equal(got, ref)
