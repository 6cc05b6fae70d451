"""FIXEDLEN frames in decompression and in the staging pass, against the CPU oracle: the words of one pass of 1024 elements on their way, or
of four, which the length of a block and the workgroups of the last round decide; blocks that end inside the first four passes, at
their edges and behind them; widths of one to 32 bits; with and without the predictor."""
import numpy as np
import pytest

import oracle
from test_gpu_reduce_k import check
from test_gpu_wave_decode import _decompress

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nz(gpu_device):
    from paper_2605_12396_amd import binding
    binding.lib()
    return binding


def _codes(n, width, seed):
    """Codes of at most `width` bits after zigzag, the widest among them in the first and the last places."""
    lim = 1 << (width - 1)
    q = np.random.default_rng(seed).integers(-lim, lim, n)
    q[[0, n - 1]] = -lim
    return q


# 16384 elements: the last block that counts as short; a block of 65536 in a grid far from full: four passes too
@pytest.mark.parametrize("predictor", [0, 1])
@pytest.mark.parametrize("width", [1, 7, 14, 21])
@pytest.mark.parametrize("n,chunk", [(2, 0), (1023, 0), (1025, 0), (4095, 0), (4096, 0), (4097, 0), (5 * 1024 + 3, 0), (3 * 16384 + 8191, 16384),
                                     (3 * 10003, 10003), (131072 + 5121, 131072 + 8192)])
def test_passes(nz, n, chunk, width, predictor):
    eb, kw = 1e-4, dict(chunk_elems=chunk, predictor=predictor)
    x = (_codes(n, width, n + width) * 1.96875e-4).astype(np.float32)
    s = oracle.compress(x, eb, oracle.make_opts(force_codec=1, **kw))[0]
    _decompress(nz, s, n, eb, **kw)
    check(nz, [s, s], n, eb, **kw)


# one workgroup a frame; 577 fill three quarters of 768
@pytest.mark.parametrize("frames", [576, 577, 768, 769])
@pytest.mark.parametrize("chunk", [16384, 17409])
def test_rounds(nz, frames, chunk):
    n, eb, kw = (frames - 1) * chunk + 5000, 1e-4, dict(chunk_elems=chunk)
    x = np.tile((_codes(1 << 18, 12, frames) * 1.96875e-4).astype(np.float32), n // (1 << 18) + 1)[:n]
    s = oracle.compress(x, eb, oracle.make_opts(force_codec=1, **kw))[0]
    _decompress(nz, s, n, eb, **kw)
    check(nz, [s, s], n, eb, **kw)
