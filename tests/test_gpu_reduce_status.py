"""What a reduce reports of broken operands, against the CPU oracle: the status of the operand, whichever it is, through passes of 256 and of 512 threads that
hand each other the worst they have seen; of several, the worst; and nothing published."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import gpu_reduce_local
from test_gpu_reduce_k import gpu_reduce_k, nz  # noqa: F401

pytestmark = pytest.mark.gpu
EB = 1e-4


def _break(s, how, frame, nf):
    """A stream with one thing wrong in `frame`: its magic, its width of a bin, or its last segments' lengths (found while decoding)."""
    t = s.copy()
    off = int(t[64 + 8 * frame:72 + 8 * frame].view(np.uint64)[0])
    h = t[off:off + 32].view(np.uint32)
    if how == "magic":
        h[0] ^= 1
    elif how == "step":
        h[6] ^= 1
        h[7] ^= 1
    else:
        nsym, nseg = int(h[4]), (nf + 255) // 256
        at = off + 32 + (nsym + 3) // 4 * 4 + 2 * (nseg - 2)
        t[at:at + 4] = (t[at:at + 4].copy().view(np.uint16) + np.array([1, 65535], np.uint16)).view(np.uint8)
    return t


# frames of three 65536-element blocks; 300001: passes of 512 threads behind a staging one of 256; 1300001: 256 for the last one too
@pytest.mark.parametrize("n", [300001, 1300001])
@pytest.mark.parametrize("k,broken", [(2, {0: "late"}), (2, {1: "late"}), (3, {0: "step"}), (3, {1: "late"}), (4, {1: "magic"}), (4, {2: "step"}), (4, {3: "late"}),
                                      (4, {0: "late", 2: "step"}), (4, {1: "step", 3: "late"}), (5, {0: "magic", 4: "step"})])
def test_reduce_k(nz, n, k, broken):  # noqa: F811
    chunk = 196608
    kw = dict(chunk_elems=chunk)
    rng = np.random.default_rng(n)
    s = oracle.compress(rng.laplace(0, 1e-3, n).astype(np.float32), EB, oracle.make_opts(force_codec=2, **kw))[0]
    frame = (n - 1) // chunk
    ops = [_break(s, broken[p], frame, n - frame * chunk) if p in broken else s for p in range(k)]
    worst = max(oracle.reduce_k([t, s], n, EB, oracle.make_opts(**kw))[2] for p, t in enumerate(ops) if p in broken)
    rc, r, _ = gpu_reduce_k(nz, ops, n, EB, nz.make_opts(**kw))
    assert rc == 0 and worst != 0 and r["status"] == worst and r["bytes"] == 0
    rc, r, got = gpu_reduce_k(nz, [s] * k, n, EB, nz.make_opts(**kw))     # (nothing of it is left in the workspace of another call)
    assert r["status"] == 0 and r["bytes"] == got.size > 0


@pytest.mark.parametrize("n", [300001, 1300001])
@pytest.mark.parametrize("how", ["magic", "step", "late"])
@pytest.mark.parametrize("first", [True, False])
def test_ring_step(nz, n, how, first):  # noqa: F811
    chunk = 196608
    kw = dict(chunk_elems=chunk)
    rng = np.random.default_rng(n + 1)
    x = rng.laplace(0, 1e-3, n).astype(np.float32)
    s = oracle.compress(x, EB, oracle.make_opts(force_codec=2, **kw))[0]
    frame = 0 if first else (n - 1) // chunk
    t = _break(s, how, frame, min(chunk, n - frame * chunk))
    want = oracle.reduce_local(t, x, EB, oracle.make_opts(**kw))[2]
    rc, r, _ = gpu_reduce_local(nz, t, x, EB, nz.make_opts(**kw))
    assert rc == 0 and want != 0 and r["status"] == want and r["bytes"] == 0
