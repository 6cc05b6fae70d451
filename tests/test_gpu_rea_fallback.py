"""Sampled path, frames of many encoder groups that are planned FIXEDLEN or HUFFMAN from their sample and fall back to RAW for what lies
behind it: one value too wide or unquantizable in the last group, in a group past the sixty-fourth, or in the first behind the sample; a
realized size past RAW, or short of the minimum gain.  The same through the ring step, whose RAW frames hold the sums of the dequantized
operands.  Against the CPU oracle; every case is one that falls back."""
import numpy as np
import pytest

from test_gpu_rea import check_rea, check_ring_rea

pytestmark = pytest.mark.gpu

EB = 1e-4


@pytest.fixture(scope="module")
def nz(gpu_device):
    from paper_2605_12396_amd import binding
    binding.lib()
    return binding


def _calm(n, chunk, seed):
    """Nothing wider than the first value of every frame."""
    x = np.clip(np.random.default_rng(seed).laplace(0, 1e-3, n), -0.004, 0.004).astype(np.float32)
    x[::chunk] = -0.004
    return x


# (elements, frame length): 256 groups of 4096 a frame, one of them ragged; 64 and 32 groups of 8192; whole groups
SHAPES = [(1 << 20, 1 << 20), ((1 << 20) - 4095, 1 << 20), (9 * 524288 + 70001, 524288), (33 * (1 << 20), 1 << 20)]
VALUES = {"wide": 5.0, "nan": np.nan, "huge": 1e30}


# (a wide value is an escape of a HUFFMAN frame: no fallback)
@pytest.mark.parametrize("force,value", [(1, "wide"), (1, "nan"), (1, "huge"), (2, "nan"), (2, "huge")])
@pytest.mark.parametrize("n,chunk", SHAPES)
def test_one_value(nz, n, chunk, force, value):
    x = _calm(n, chunk, n % 1009)
    last = n - (n - 1) // chunk * chunk
    at = [chunk * f + p for f, p in ((0, min(n, chunk) - 1), (0, 70 * 4096 + 3), (0, 16384), ((n - 1) // chunk, last - 1))]
    for i, where in enumerate(at[:2] if n > 1 << 23 else at):
        y = x.copy()
        y[where] = VALUES[value]
        _, ores, _, _, _ = check_rea(nz, y, EB, cal=x[:65536], chunk_elems=chunk, force_codec=force)
        assert ores.n_fallback == 1, (i, where)


def _late(n, chunk, seed, share, behind):
    """Calm frames with a share of escapes from element `behind` of each frame on."""
    x, rng = _calm(n, chunk, seed), np.random.default_rng(seed + 1)
    hit = (np.arange(n) % chunk >= behind) & (rng.random(n) < share)
    x[hit] = rng.uniform(-3, 3, int(hit.sum()))
    return x


# all of the frame behind the sample escapes: past the RAW size; a third of it: short of a gain of 600 in a thousand
@pytest.mark.parametrize("share,gain", [(1.0, 0), (0.35, 600)], ids=["realized", "gain"])
@pytest.mark.parametrize("n,chunk", SHAPES[:3])
def test_size(nz, n, chunk, share, gain):
    x = _late(n, chunk, 5, share, 16384)
    _, ores, _, _, _ = check_rea(nz, x, EB, cal=x[:16384], chunk_elems=chunk, force_codec=2 if not gain else -1, min_gain_permil=gain)
    assert ores.n_fallback == ores.n_frames


@pytest.mark.parametrize("what", ["wide", "realized", "gain"])
@pytest.mark.parametrize("n,chunk", SHAPES[:3])
def test_ring_step(nz, n, chunk, what):
    a, x, kw = _calm(n, chunk, 21), _calm(n, chunk, 22), dict(chunk_elems=chunk)
    if what == "wide":
        x[[70 * 4096 + 3, n - 1]] = 5.0
        kw["force_codec"] = 1
    else:
        x = _late(n, chunk, 23, 1.0 if what == "realized" else 0.35, 16384)
        kw.update(dict(force_codec=2) if what == "realized" else dict(min_gain_permil=600))
    ores = check_ring_rea(nz, a, x, EB, a_kw=dict(chunk_elems=chunk), **kw)[1]
    if what == "wide":
        assert ores.n_fallback == len({(70 * 4096 + 3) // chunk, (n - 1) // chunk})
    else:
        assert ores.n_fallback >= max(1, ores.n_frames - 1)        # (a short last frame may still fit)
