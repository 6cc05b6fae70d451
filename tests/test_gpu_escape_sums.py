"""GPU parity of the adding passes over HUFFMAN frames in which escapes are frequent, against the CPU oracle: the reader
reloads its window at escapes, in every place of a run of eight symbols and of a phase, up to segments of nothing but
escapes, at the edges of segments, halves and blocks.  Bytes have to be the same."""
import numpy as np
import pytest

import oracle
from test_gpu_reduce_k import check

pytestmark = pytest.mark.gpu

SHAPES = [(7, 0), (257, 0), (65536, 65536), (65536 + 2047, 0), (131072 + 2050, 262144), (3 * 10003, 10003)]


@pytest.fixture(scope="module")
def nz(gpu_device):
    from paper_2605_12396_amd import binding
    binding.lib()
    return binding


def _message(n, share, seed):
    """Codes of a few bits, `share` of the elements far outside the alphabet, and one run of 600 of those."""
    rng = np.random.default_rng(seed)
    x = rng.laplace(0, 2e-3, n)
    far = rng.random(n) < share
    x[far] = rng.uniform(-1, 1, int(far.sum()))
    x[n // 3:n // 3 + 600] = rng.uniform(0.5, 1, x[n // 3:n // 3 + 600].size)
    return x.astype(np.float32)


@pytest.mark.parametrize("share", [0.005, 0.08, 0.5, 1.0])
@pytest.mark.parametrize("n,chunk", SHAPES)
def test_escapes(nz, n, chunk, share):
    import torch
    eb, kw = 1e-4, dict(chunk_elems=chunk)
    o, of = oracle.make_opts(**kw), oracle.make_opts(force_codec=2, **kw)
    xs = [_message(n, share, 40 + p) for p in range(3)]
    ss = [oracle.compress(x, eb, of)[0] for x in xs]
    check(nz, ss[:2], n, eb, **kw)
    check(nz, ss, n, eb, **kw)
    ref, ores, orc = oracle.reduce_local(ss[0], xs[1], eb, o)
    sess = nz.Session(n, nz.make_opts(**kw), "cuda:0", reduce=True)
    ds = torch.from_numpy(np.concatenate([ss[0], np.zeros((-ss[0].size) % 16, np.uint8)])).to("cuda:0")
    rc, out = sess.reduce_local(ds, ss[0].size, torch.from_numpy(xs[1]).to("cuda:0"), n, eb)
    r = sess.result()
    assert rc == 0 and orc == 0 and r["status"] == 0 and r["bytes"] == ores.bytes
    assert np.array_equal(out[:r["bytes"]].cpu().numpy(), ref)
