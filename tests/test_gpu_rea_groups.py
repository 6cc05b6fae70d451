"""GPU parity of the sampled path where its encoder groups follow the size of the message, against the CPU oracle: every group size,
ragged ends of one symbol to one short of a group, words in which groups meet, frames that are FIXEDLEN or RAW by plan, and
the ring step (frames that fall back: test_gpu_rea_fallback.py).  Bytes, plans and result records have to be the same."""
import numpy as np
import pytest

from test_gpu_rea import check_rea, check_ring_rea

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nz(gpu_device):
    from paper_2605_12396_amd import binding
    binding.lib()
    return binding


def _message(kind, n, seed):
    rng = np.random.default_rng(seed)
    if kind == "flat":
        return rng.uniform(-1, 1, n).astype(np.float32)
    x = rng.laplace(0, 1e-3, n)
    if kind == "escapes":
        at = rng.random(n) < 0.1
        x[at] = rng.uniform(-3, 3, int(at.sum()))
    return x.astype(np.float32)


# groups of 4096, 8192, 16384 and 32768 symbols, and whole ones; the ends: a whole group, one symbol, one short of a group
SIZES = [(65537, 65537), (262144 + 1, 262144), (300007, 0), (3 * 100000 - 1, 100000), ((1 << 21) + 4096, 1 << 20), (512 * 4096 + 1, 0),
         (512 * 8192 - 8191, 1 << 20), (511 * 16384 + 31, 0), (512 * 32768 + 77, 0)]


@pytest.mark.parametrize("kind", ["laplace", "flat", "escapes"])
@pytest.mark.parametrize("n,chunk", SIZES)
def test_group_sizes(nz, n, chunk, kind):
    check_rea(nz, _message(kind, n, n % 1000), 1e-4, chunk_elems=chunk)


@pytest.mark.parametrize("force", [0, 1, 2])
@pytest.mark.parametrize("n,chunk", [(65536 + 4097, 0), (300007, 100000)])
def test_pinned_codecs(nz, n, chunk, force):
    check_rea(nz, _message("escapes", n, 3), 1e-4, chunk_elems=chunk, force_codec=force)


@pytest.mark.parametrize("kind", ["laplace", "flat", "escapes"])
@pytest.mark.parametrize("n,chunk", [(65537, 65537), (300007, 0), (512 * 4096 + 1, 1 << 20), (511 * 16384 + 31, 0)])
def test_ring_step(nz, n, chunk, kind):
    check_ring_rea(nz, _message(kind, n, 11), _message(kind, n, 12), 1e-4, chunk_elems=chunk)
