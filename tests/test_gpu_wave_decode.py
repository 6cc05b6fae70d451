"""GPU parity of the HUFFMAN decoder where its steps of two lookups can go wrong, against the CPU oracle: codes longer than the
first-level table and escapes at the edges of segments, phases of 32 symbols and steps of up to four (a lane that has what it needs
must not read on), one behind the other, and codes past 17 bits; with and without the predictor; and the workgroups of 512
threads that large messages take, with frames that they fill in part.  Values and bytes have to be the same."""
import numpy as np
import pytest

import oracle
from crafted import incomplete_code_stream
from test_gpu_reduce_k import check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nz(gpu_device):
    from paper_2605_12396_amd import binding
    binding.lib()
    return binding


def _decompress(nz, stream, n, eb, **kw):
    import torch
    sess = nz.Session(n, nz.make_opts(**kw), "cuda:0", reduce=False)
    ds = torch.from_numpy(np.concatenate([stream, np.zeros((-stream.size) % 16, np.uint8)])).to("cuda:0")
    rc, y = sess.decompress(ds, stream.size, n, eb)
    assert rc == 0 and sess.result()["status"] == 0
    ref, ores, orc = oracle.decompress(stream, n, eb)
    assert orc == 0
    assert np.array_equal(y.cpu().numpy().view(np.uint32), ref.view(np.uint32))


def _placed(n, what, period, phase, seed):
    """Codes of two or three bits, and at every `period`-th place from `phase` on a rare symbol, an escape, or either."""
    rng = np.random.default_rng(seed)
    q = rng.integers(-2, 3, n)
    at = np.arange(phase, n, period)
    rare = rng.integers(20, 120, at.size) * rng.choice([-1, 1], at.size)       # some 200 symbols share a percent or less
    far = rng.integers(200, 30000, at.size)
    q[at] = rare if what == "long" else far if what == "escape" else np.where(rng.random(at.size) < 0.5, rare, far)
    return (q * 1.96875e-4).astype(np.float32)


@pytest.mark.parametrize("predictor", [0, 1])
@pytest.mark.parametrize("what,period", [("long", 256), ("long", 32), ("escape", 256), ("escape", 4), ("both", 33), ("both", 2)])
@pytest.mark.parametrize("phase", [0, 1, 31, 255])
def test_edges(nz, what, period, phase, predictor):
    n, eb, kw = 65536 + 4133, 1e-4, dict(chunk_elems=65536, predictor=predictor)
    x = _placed(n, what, period, phase, 7 * period + phase)
    s = oracle.compress(x, eb, oracle.make_opts(force_codec=2, **kw))[0]
    _decompress(nz, s, n, eb, **kw)
    check(nz, [s, s], n, eb, **kw)


@pytest.mark.parametrize("predictor", [0, 1])
def test_deep_codes(nz, predictor):
    """Counts that halve from symbol to symbol: code lengths up to 17 and past it under one 11-bit prefix."""
    n, eb, kw = 262144, 1e-4, dict(chunk_elems=262144, predictor=predictor)
    rng = np.random.default_rng(5)
    z = np.minimum(np.floor(-np.log2(1.0 - rng.random(n))).astype(np.int64), 40)
    q = np.where(z & 1, -(z + 1) // 2, z // 2)
    q[rng.integers(0, n, 40)] = 5000
    x = (np.cumsum(q) % 30000 if predictor else q) * 1.96875e-4
    s = oracle.compress(x.astype(np.float32), eb, oracle.make_opts(force_codec=2, **kw))[0]
    _decompress(nz, s, n, eb, **kw)
    check(nz, [s, s, s], n, eb, **kw)


@pytest.mark.parametrize("frames,chunk", [(384, 65537), (385, 65537), (385, 98304 + 2), (386, 131071)])
def test_width_of_workgroups(nz, frames, chunk):
    """768 blocks of 65536 take workgroups of 256 threads, the next ones 512: frames of two blocks that fill the second in part, and a
    ragged last frame (the rest of the rule: test_gpu_dec_width.py)."""
    n = (frames - 1) * chunk + chunk // 3 + 1
    eb, kw = 1e-5, dict(chunk_elems=chunk)
    x = np.random.default_rng(frames).laplace(0, 1e-3, 1 << 20).astype(np.float32)
    x = np.tile(x, n // x.size + 1)[:n]
    s = oracle.compress(x, eb, oracle.make_opts(**kw))[0]
    _decompress(nz, s, n, eb, **kw)
    check(nz, [s, s], n, eb, **kw)


@pytest.mark.parametrize("bits_per_symbol", [1, 8])
@pytest.mark.parametrize("op", ["decompress", "reduce", "ring"])
def test_bits_that_start_no_code(nz, op, bits_per_symbol):
    """The only code is the bit 0.  A 1 and what follows it are looked up in both tables and found in neither; where the 1 is the last
    lookup of a run, the windows of the next runs are requested between the two (8 bits a symbol), and its lane may not
    come out behind them.  Segment s of a frame has its first 1 at bit s, so that every place of a phase is one's last lookup."""
    from test_gpu_parity import gpu_decompress, gpu_reduce, gpu_reduce_local
    eb = 1e-4
    step_bits = int(np.float32(oracle.step_constants(eb)[0]).view(np.uint32))
    for n, every in ((256 * 256, 0), (256 * 256, 41), (3 * 256 + 77, 29)):
        segs = np.arange((n + 255) // 256)
        at = (256 * segs * bits_per_symbol + segs)[segs < bits_per_symbol * np.minimum(256, n - 256 * segs)]
        if every:
            at = np.concatenate([at, np.arange(13, n * bits_per_symbol, every)])
        bad = incomplete_code_stream(n, step_bits, at, bits_per_symbol)
        good = oracle.compress(np.random.default_rng(n).laplace(0, 1e-3, n).astype(np.float32), eb, oracle.make_opts(chunk_elems=n))[0]
        g, o, x = nz.make_opts(chunk_elems=n), oracle.make_opts(chunk_elems=n), np.zeros(n, np.float32)
        if op == "decompress":
            ref, _, orc = oracle.decompress(bad, n, eb)
            _, r, got = gpu_decompress(nz, bad, n, eb, g)
            assert orc == oracle.ERR_CORRUPT and r["status"] == nz.ERR_CORRUPT and not ref.any() and not got.any()
        elif op == "reduce":
            for a, b in ((bad, good), (good, bad)):
                assert oracle.reduce_frames(a, b, n, eb, o)[2] == gpu_reduce(nz, a, b, n, eb, g)[1]["status"] == nz.ERR_CORRUPT
        else:
            assert oracle.reduce_local(bad, x, eb, o)[2] == gpu_reduce_local(nz, bad, x, eb, g)[1]["status"] == nz.ERR_CORRUPT
