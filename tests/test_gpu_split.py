"""GPU parity of the calls whose work split follows the size of the message, against the CPU oracle, at the sizes where
a split can go wrong: one block of every granularity, one element more or less, blocks that end in the middle of a
segment, frames that are no whole number of blocks, both ends of the alphabets, more blocks in a frame than a wavefront
has lanes, and frames of every codec side by side."""
import numpy as np
import pytest

import oracle
from paper_2605_12396_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [(1, 0), (255, 0), (4095, 0), (4096, 0), (4097, 0), (8192, 16384), (16385, 0), (32769, 16384), (65535, 0), (65536, 0),
          (65537, 65536), (131073, 0), (262144 + 3, 0), (300007, 0), (5 * 10003 + 1, 10003), (200001, 24577), (1048576, 1048576),
          (1048576 - 4095, 1048576), (700001, 524288), (2500001, 0)]


@pytest.fixture(scope="module")
def nz(gpu_device):
    from paper_2605_12396_amd import binding
    binding.lib()
    return binding


def _dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


def _message(n, seed):
    """Laplace values; stretches of zeros, of values past the alphabet, of values past 16-bit sums, and a NaN."""
    x = W.gradient_like(n, seed=seed)
    if n > 40000:
        x[20000:30000] = 0.0
        x[n // 2:n // 2 + 3000] = np.linspace(-2.0, 2.0, 3000, dtype=np.float32)
        x[n - 700:n - 100] *= 1000.0
        if seed % 3 == 0:
            x[n // 3] = np.nan
    return x


def _kw(i):
    return [dict(), dict(alphabet=1024), dict(alphabet=2), dict(alphabet=512), dict(predictor=1)][i]


@pytest.mark.parametrize("variant", range(5))
@pytest.mark.parametrize("n,chunk", SHAPES)
def test_compress(nz, n, chunk, variant):
    kw, eb = dict(_kw(variant), chunk_elems=chunk), 1e-4
    x = _message(n, 7 + n + variant)
    sess = nz.Session(n, nz.make_opts(**kw), "cuda:0")
    ref, ores, orc = oracle.compress(x, eb, oracle.make_opts(**kw))
    rc, out = sess.compress(_dev(x), eb)
    r = sess.result()
    assert rc == 0 and orc == 0 and r["status"] == 0 and r["bytes"] == ores.bytes
    assert (r["n_raw"], r["n_fixed"], r["n_huff"]) == (ores.n_raw, ores.n_fixed, ores.n_huff)
    assert np.array_equal(out[:r["bytes"]].cpu().numpy(), ref)


@pytest.mark.parametrize("n,chunk", SHAPES[3::3])
def test_compress_stochastic(nz, n, chunk):
    import torch
    x, step = _message(n, 5), 2e-4
    g, o = nz.make_opts(chunk_elems=chunk), oracle.make_opts(chunk_elems=chunk)
    sess = nz.Session(n, g, "cuda:0")
    out = sess.new_stream_buffer()
    assert nz.nz_compress_sr(_dev(x), n, step, 99, out, sess.cap, sess.res, g, sess.ws, sess.ws_bytes) == 0
    ref, ores, orc = oracle.compress_sr(x, np.float32(step), 99, o)
    r = sess.result()
    assert orc == 0 and r["status"] == 0 and r["bytes"] == ores.bytes
    assert np.array_equal(out[:r["bytes"]].cpu().numpy(), ref)
    torch.cuda.synchronize()
