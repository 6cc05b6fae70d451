"""Ring steps whose own data in a frame cannot be quantized, against the CPU oracle, byte for byte: the frame turns RAW after its sums have been staged, in
parts that other workgroups have staged; from incoming codes and from incoming RAW words; with the output apart from the operands and on top of either, where
both have to be read before anything is written."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import gpu_reduce_local
from test_gpu_sr import _gpu_reduce_local_sr, nz  # noqa: F401

pytestmark = pytest.mark.gpu
EB = 1e-4


def _messages(n, chunk, incoming):
    rng = np.random.default_rng(n)
    a, x = (rng.laplace(0, 1e-3, n).astype(np.float32) for _ in range(2))
    x[3], x[n // 2], x[n - 1] = 5.0, 40000 * 2e-4, np.nan               # (a wide code; frames that cannot be quantized)
    x[min(n - 2, 2 * chunk - 1)] = np.inf
    if incoming == "raw":
        a[[0, n // 2, n - 1]] = np.nan, np.inf, 1e30                     # RAW on both sides, or on one
    return a, x


@pytest.mark.parametrize("incoming", ["coded", "raw"])
@pytest.mark.parametrize("n,chunk", [(5, 16), (70001, 65536), (3 * 65536 + 7, 1 << 20), (2 * 262144 + 70001, 262144), (5 * 16384 + 5, 16384), (3 * 10001, 10001)])
@pytest.mark.parametrize("predictor", [0, 1])
def test_values_that_cannot_be_quantized(nz, n, chunk, predictor, incoming):  # noqa: F811
    a, x = _messages(n, chunk, incoming)
    kw = dict(chunk_elems=chunk, predictor=predictor)
    s = oracle.compress(a, EB, oracle.make_opts(**kw))[0]
    ref, ores, orc = oracle.reduce_local(s, x, EB, oracle.make_opts(**kw))
    rc, r, got = gpu_reduce_local(nz, s, x, EB, nz.make_opts(**kw))
    assert rc == 0 and orc == 0 and r["status"] == 0 and r["n_raw"] == ores.n_raw > 0
    assert r["bytes"] == ores.bytes and np.array_equal(got, ref)


@pytest.mark.parametrize("on", ["incoming", "local"])
@pytest.mark.parametrize("incoming", ["coded", "raw"])
@pytest.mark.parametrize("n,chunk", [(70001, 65536), (2 * 262144 + 70001, 262144), (40 * 16384 + 5, 16384)])
def test_output_on_an_operand(nz, n, chunk, incoming, on):  # noqa: F811
    import torch
    a, x = _messages(n, chunk, incoming)
    g, o = nz.make_opts(chunk_elems=chunk), oracle.make_opts(chunk_elems=chunk)
    s = oracle.compress(a, EB, o)[0]
    ref, ores, _ = oracle.reduce_local(s, x, EB, o)
    sess = nz.Session(n, g, "cuda:0", reduce=True)
    out = torch.zeros(sess.cap, dtype=torch.uint8, device="cuda:0")
    incoming_d, local_d = torch.from_numpy(s).cuda(), torch.from_numpy(x).cuda()
    if on == "incoming":
        out[:s.size] = incoming_d
        incoming_d = out
    else:
        out[:4 * n].view(torch.float32)[:] = local_d
        local_d = out[:4 * n].view(torch.float32)
    rc = nz.nz_reduce_local(incoming_d, s.size, local_d, out, sess.cap, n, EB, sess.res, g, sess.ws, sess.ws_bytes)
    r = sess.result()
    assert rc == 0 and r["status"] == 0 and r["bytes"] == ores.bytes
    assert np.array_equal(out[:r["bytes"]].cpu().numpy(), ref)


@pytest.mark.parametrize("incoming", ["coded", "raw"])
def test_stochastic(nz, incoming):  # noqa: F811
    n, chunk, step = 2 * 262144 + 70001, 262144, 2e-4
    a, x = _messages(n, chunk, incoming)
    o, g = oracle.make_opts(chunk_elems=chunk), nz.make_opts(chunk_elems=chunk)
    s = oracle.compress_sr(a, step, 7, o)[0]
    ref, ores, orc = oracle.reduce_local_sr(s, x, step, 9, o)
    rc, r, got = _gpu_reduce_local_sr(nz, s, x, step, 9, g)
    assert rc == 0 and orc == 0 and r["status"] == 0 and r["n_raw"] == ores.n_raw > 0
    assert r["bytes"] == ores.bytes and np.array_equal(got, ref)
