"""GPU parity of the HUFFMAN decoder's steps, against the CPU oracle, for every kind of frame that they tell apart: one that is all pairs of short
codes, pairs with and without escapes, windows renewed once a phase and every few steps, segments that outrun theirs, no codes of more than 11 bits, alphabets
whose codes have two bytes; with messages that end anywhere in a segment's phases, where a step must not take a symbol too many; and
streams of differences, whose escapes are the segments' first symbols or others too."""
import numpy as np
import pytest

import oracle
from test_gpu_reduce_k import check
from test_gpu_wave_decode import _decompress, nz  # noqa: F401

pytestmark = pytest.mark.gpu


def _codes(kind, n, seed):
    rng = np.random.default_rng(seed)
    if kind == "two bits":
        return rng.integers(-1, 2, n)
    if kind == "flat":                                           # 199 symbols, equally likely: seven and eight bits, no escape
        return rng.integers(-99, 100, n)
    scale = {"short": 5.0, "some escapes": 2.0, "middle": 15.0, "six bits": 10.0, "uneven": 1.5, "long": 50.0}[kind]
    q = np.rint(rng.laplace(0.0, scale, n)).astype(np.int64)
    if kind == "uneven":                                         # one segment in nine of eleven bits and more, which outruns its windows; no escape
        q = np.where(np.arange(n) // 256 % 9 == 4, rng.integers(-120, 121, n), q)
    if kind == "some escapes":
        q = np.where(rng.random(n) < 0.01, rng.integers(-20000, 20000, n), q)
    return np.clip(q, -32000, 32000)


@pytest.mark.parametrize("alphabet", [0, 512, 1024])
@pytest.mark.parametrize("kind", ["two bits", "short", "some escapes", "middle", "six bits", "uneven", "flat", "long"])
@pytest.mark.parametrize("n", [1, 35, 256 + 3, 256 * 64 + 36, 65536 + 256 * 7 + 225, 131072 + 33])
def test_kinds(nz, n, kind, alphabet):  # noqa: F811
    eb, kw = 1e-4, dict(alphabet=alphabet, chunk_elems=65536 if n % 2 else 0)
    streams = [oracle.compress((_codes(kind, n, 11 * n + s) * 1.96875e-4).astype(np.float32), eb, oracle.make_opts(force_codec=2, **kw))[0]
               for s in range(2)]
    _decompress(nz, streams[0], n, eb, **kw)
    check(nz, streams, n, eb, **kw)


@pytest.mark.parametrize("alphabet", [0, 512])
@pytest.mark.parametrize("kind", ["two bits", "short", "some escapes", "middle", "uneven", "long"])
@pytest.mark.parametrize("predictor", [0, 1])
def test_ends(nz, kind, predictor, alphabet):  # noqa: F811
    """Every number of symbols that a last segment can leave for its last phase of 32, and for the one before."""
    eb, kw = 1e-4, dict(alphabet=alphabet, predictor=predictor)
    q = _codes(kind, 4 * 256 + 100, 5)
    if predictor:                                                # (differences of that kind)
        q = np.cumsum(q - np.rint(q.mean()).astype(np.int64)) % 60000 - 30000
    x = (q * 1.96875e-4).astype(np.float32)
    for n in range(4 * 256 + 60, 4 * 256 + 96):
        s = oracle.compress(x[:n], eb, oracle.make_opts(force_codec=2, **kw))[0]
        _decompress(nz, s, n, eb, **kw)
        check(nz, [s, s], n, eb, **kw)


@pytest.mark.parametrize("alphabet", [0, 1024])
@pytest.mark.parametrize("jumps", [0.0, 3e-4, 1e-2])
@pytest.mark.parametrize("n", [37, 256 * 5 + 3, 65536 + 256 * 7 + 225, 131072 + 33])
@pytest.mark.parametrize("level", [0, 9000])
def test_differences(nz, n, level, jumps, alphabet):  # noqa: F811
    """The predictor: segments whose first symbol alone is an escape (a line far from zero) or not, and lines with some or many more."""
    rng = np.random.default_rng(n + level)
    q = level + np.cumsum(np.rint(rng.normal(0.0, 7.0, n)).astype(np.int64)) + np.where(rng.random(n) < jumps, 4000, 0)
    eb, kw = 1e-4, dict(alphabet=alphabet, predictor=1, chunk_elems=65536 if n % 2 else 0)
    s = oracle.compress((q * 1.96875e-4).astype(np.float32), eb, oracle.make_opts(force_codec=2, **kw))[0]
    _decompress(nz, s, n, eb, **kw)
    check(nz, [s, s], n, eb, **kw)
