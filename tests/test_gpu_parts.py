"""GPU parity of a reduce's encoder where its workgroups take parts of a statistics block, against the CPU oracle: every size of part,
ragged ends of one symbol to one short of a part, the words in which parts and blocks meet, escapes on both sides of them, sums
of more than 16 bits, RAW and FIXEDLEN frames, with and without the predictor.  Bytes have to be the same."""
import numpy as np
import pytest

import oracle
from test_gpu_reduce_k import check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nz(gpu_device):
    from paper_2605_12396_amd import binding
    binding.lib()
    return binding


def _message(kind, n, seed):
    """`escapes`: in every tenth place, and in the 40 places around every multiple of 4096; `wide`: sums past 16 bits there."""
    rng = np.random.default_rng(seed)
    if kind == "flat":
        return rng.uniform(-1, 1, n).astype(np.float32)
    x = rng.laplace(0, 1e-3, n)
    if kind != "laplace":
        i = np.arange(n)
        at = ((i + 20) % 4096 < 40) | (rng.random(n) < 0.1)
        x[at] = rng.uniform(2, 6.4, int(at.sum())) * (rng.choice([-1, 1], int(at.sum())) if kind == "escapes" else 1.0)
    return x.astype(np.float32)


# parts of 4096, 8192, 16384 and 32768 symbols and whole blocks: one to 64 frames' worth, and around 1024 parts
SIZES = [(4097, 0), (65536 + 1, 65536), (2 * 65536 + 8191, 0), (3 * 100003, 100003), ((1 << 20) + 4096, 1 << 20),
         (1024 * 4096, 0), (1024 * 4096 + 1, 0), (1000 * 8192 - 31, 1 << 20), (1024 * 16384 + 1, 0)]


@pytest.mark.parametrize("kind", ["laplace", "flat", "escapes", "wide"])
@pytest.mark.parametrize("n,chunk", SIZES)
def test_sum_of_two(nz, n, chunk, kind):
    eb, kw = 1e-4, dict(chunk_elems=chunk)
    ss = [oracle.compress(_message(kind, n, 5 + p), eb, oracle.make_opts(**kw))[0] for p in range(2)]
    check(nz, ss, n, eb, **kw)


@pytest.mark.parametrize("force", [0, 1, 2])
@pytest.mark.parametrize("predictor", [0, 1])
@pytest.mark.parametrize("n,chunk", [(65536 + 4099, 0), (3 * 100003, 100003), (2 * 65536 + 8191, 0)])
def test_pinned_codecs(nz, n, chunk, predictor, force):
    eb, kw = 1e-4, dict(chunk_elems=chunk, predictor=predictor)
    ss = [oracle.compress(_message("escapes", n, 9 + p), eb, oracle.make_opts(**kw))[0] for p in range(2)]
    check(nz, ss, n, eb, force_codec=force, **kw)


@pytest.mark.parametrize("alphabet", [2, 16, 1024])
def test_alphabets(nz, alphabet):
    n, eb, kw = 3 * 65536 + 4095, 1e-4, dict(chunk_elems=0, alphabet=alphabet)
    ss = [oracle.compress(_message("laplace", n, 15 + p), eb, oracle.make_opts(**kw))[0] for p in range(2)]
    check(nz, ss, n, eb, **kw)
