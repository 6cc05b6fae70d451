"""HUFFMAN frames whose length is no multiple of four, so that most of them start off one: decompression, the sums and the ring step take
their codes four at a time there too, with the last ones of a frame one by one.  Against the CPU oracle, at the edges of a
wavefront's rows, of halves and of blocks; with the predictor, with codes and sums past 16 bits, and with local values that cannot be quantized."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import gpu_reduce_local
from test_gpu_rea import check_ring_rea
from test_gpu_reduce_k import check
from test_gpu_sr import _gpu_reduce_local_sr
from test_gpu_wave_decode import _decompress, _placed

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nz(gpu_device):
    from paper_2605_12396_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("kind", ["", "wide", "predictor", "unquantizable"])
@pytest.mark.parametrize("chunk", [5, 255, 8191, 16385, 16387, 65537, 131071, 131074])
def test_odd_frames(nz, chunk, kind):
    n, eb = 5 * chunk + chunk // 2 + 1, 1e-4
    kw = dict(chunk_elems=chunk, predictor=int(kind == "predictor"))
    a, x = (_placed(n, "both", 61, p, chunk + p) for p in (3, 7))
    if kind == "wide":                                             # an operand's code, a local one and a sum of more than 16 bits
        a[[0, n // 2, n - 1]], x[[1, n // 3, n - 1]] = 8.0, -9.0
        a[n // 4], x[n // 4] = 5.0, 5.0
    o, of = oracle.make_opts(**kw), oracle.make_opts(force_codec=2, **kw)
    s = oracle.compress(a, eb, of)[0]
    _decompress(nz, s, n, eb, **kw)
    check(nz, [s, oracle.compress(x, eb, of)[0], s], n, eb, **kw)
    if kind == "unquantizable":
        x[[n // 5, n - 1]] = np.nan, 1e9
    ref, ores, orc = oracle.reduce_local(s, x, eb, o)
    _, r, got = gpu_reduce_local(nz, s, x, eb, nz.make_opts(**kw))
    assert orc == 0 and r["status"] == 0 and r["bytes"] == ores.bytes and np.array_equal(got, ref)
    if kind != "predictor":
        check_ring_rea(nz, a, x, eb, a_kw=dict(force_codec=2, **kw), **kw)
        step = float(np.float32(2e-4))
        ss = oracle.compress_sr(a, step, 7, of)[0]
        ref, ores, orc = oracle.reduce_local_sr(ss, x, step, 8, o)
        _, r, got = _gpu_reduce_local_sr(nz, ss, x, step, 8, nz.make_opts(**kw))
        assert orc == 0 and r["status"] == 0 and r["bytes"] == ores.bytes and np.array_equal(got, ref)
