"""Decompression and staging on both sides of the rule for the width of their workgroups, against the CPU oracle: 512 threads where they
make one round of workgroups of two, and two rounds of three unless the stream has four to twelve bits a symbol; frames of two
blocks, the second filled in part, and a ragged last frame; and frames that are found broken in their last workgroup's share, which
are cleared as a whole by the pass behind."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import gpu_decompress
from test_gpu_reduce_k import check

pytestmark = pytest.mark.gpu

CHUNK = 65536 + 20002


@pytest.fixture(scope="module")
def nz(gpu_device):
    from paper_2605_12396_amd import binding
    binding.lib()
    return binding


def _stream(n, kind, kw):
    rng = np.random.default_rng(n)
    x = rng.uniform(-1, 1, 1 << 18) if kind == "fixed" else rng.laplace(0, 1e-3, 1 << 18) if kind == "dense" else 4e-4 * (rng.random(1 << 18) < 0.1)
    eb = 1e-5 if kind == "dense" else 1e-4
    s, _, rc = oracle.compress(np.tile(x.astype(np.float32), n // x.size + 1)[:n], eb, oracle.make_opts(force_codec=1 if kind == "fixed" else 2, **kw))
    bits = 8 * s.size / n
    assert rc == 0 and (bits < 4 if kind == "short" else 12 <= bits < 32 if kind == "fixed" else 4 <= bits < 12)
    return s, eb


# two blocks a frame: 768 blocks are one round of 256 threads, 1024 one of 512, 1536 two of 256, 2048 two of 512
@pytest.mark.parametrize("kind", ["short", "dense", "fixed"])
@pytest.mark.parametrize("frames", [385, 512, 513, 769])
def test_decompress(nz, frames, kind):
    n, kw = (frames - 1) * CHUNK + 70001, dict(chunk_elems=CHUNK)
    s, eb = _stream(n, kind, kw)
    offs = s[64:64 + 8 * frames].view(np.uint64)
    broken = s.copy()
    for f in (3, frames // 2, frames - 1) if kind != "fixed" else ():  # a bit of the last segment counts for the one before it
        nseg = (min(CHUNK, n - f * CHUNK) + 255) // 256
        lengths = int(s[int(offs[f]) + 16:int(offs[f]) + 20].view(np.uint32)[0])
        at = int(offs[f]) + 32 + (lengths + 3) // 4 * 4 + 2 * (nseg - 2)
        broken[at:at + 4] = (s[at:at + 4].copy().view(np.uint16) + np.array([1, 65535], np.uint16)).view(np.uint8)
    for t in (s, broken) if kind != "fixed" else (s,):
        ref, ores, orc = oracle.decompress(t, n, eb)
        _, r, got = gpu_decompress(nz, t, n, eb, nz.make_opts(**kw))
        assert r["status"] == orc and (t is s) == (orc == 0)
        assert (r["n_raw"], r["n_fixed"], r["n_huff"]) == (ores.n_raw, ores.n_fixed, ores.n_huff)
        assert np.array_equal(got.view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("kind", ["short", "dense", "fixed"])
def test_staging(nz, kind):
    frames, kw = 769, dict(chunk_elems=CHUNK)
    n = (frames - 1) * CHUNK + 70001
    s, eb = _stream(n, kind, kw)
    check(nz, [s, s], n, eb, **kw)


def _codes(kind, n):
    """Codes of 256 Ki elements, repeated."""
    rng = np.random.default_rng(n)
    m = 1 << 18
    if kind == "rare":                                                   # four heavy symbols, a thousand rare ones: more prefixes of long codes than tables
        q = np.where(rng.random(m) < 0.9, rng.integers(-2, 2, m), rng.integers(-505, 506, m))
    elif kind == "line":                                                 # (predictor) differences that are small but for a segment's first, and some that are not
        q = np.cumsum(rng.integers(-6, 7, m)) % 20000 - 10000
        q = np.where(rng.random(m) < 1e-3, -q, q)
    else:
        q = np.rint(rng.laplace(0, {"long": 50.0, "short": 5.0}[kind], m)).astype(np.int64)
    return np.tile((np.clip(q, -32000, 32000) * 1.96875e-4).astype(np.float32), n // m + 1)[:n]


@pytest.mark.parametrize("kind,alphabet", [("rare", 1024), ("long", 1024), ("short", 1024), ("long", 512), ("line", 0), ("line", 1024)])
@pytest.mark.parametrize("frames", [3, 512])
def test_codes_of_two_bytes_and_differences(nz, frames, kind, alphabet):
    """Both widths, with alphabets whose kernels are their own and with the predictor: two blocks a frame, the last one ragged."""
    n, kw = (frames - 1) * CHUNK + 70001, dict(chunk_elems=CHUNK, alphabet=alphabet, predictor=1 if kind == "line" else 0)
    s, _, rc = oracle.compress(_codes(kind, n), 1e-4, oracle.make_opts(force_codec=2, **kw))
    ref, _, orc = oracle.decompress(s, n, 1e-4)
    _, r, got = gpu_decompress(nz, s, n, 1e-4, nz.make_opts(**kw))
    assert rc == 0 and orc == 0 and r["status"] == 0 and r["n_huff"] == frames
    assert np.array_equal(got.view(np.uint32), ref.view(np.uint32))
    if frames == 3 or kind in ("rare", "line"):
        check(nz, [s] * 3, n, 1e-4, **kw)
