"""The tile kernel with one workgroup per CU at every tile height it can have (1 to 16 slabs of 16 rows, with and without
chunks of one slab more), several rounds of tiles per workgroup, and K steps fewer than, as many as and more than the stages of
its LDS ring: the first and last row of every slab against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2305_10727_amd import synth
from test_gpu_parity import dev, fp16_problem, g, force_kernel, host, rel_err, ulp_diff_f16, _oracle_weights  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (on 256 CUs; 1024 channels: 64 chunks to a round) one round of each height, the last with a part of a slab, and two
# of chunks of two heights; whole rounds of the highest tiles with a tail behind them; then rounds of 2 and 3, the last tile partly
# outside Y, and channels that are no whole lines
SHAPES = [(1024 * h - 5, (128, 256, 384, 512, 640, 768)[h % 6], 1024) for h in range(1, 17)]
SHAPES += [(1024 * h + 70, (640, 128, 512, 384)[h % 4], 1024) for h in (1, 3, 4, 8, 11, 12, 15)]
SHAPES += [(13556, 512, 5120)]
SHAPES += [(51 * 256 * 3 + 300, 128, 1280), (20000, 128, 1024), (20000, 512, 1024), (12608, 768, 1000), (30000, 256, 264), (12608, 128, 300), (5000, 384, 4)]


def _rows(M):
    m = np.arange(M)
    return m[(m % 16 == 0) | (m % 16 == 15) | (m == M - 1)]


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_int8(g, force_kernel, M, K, N):
    force_kernel(2)
    rng = np.random.default_rng(M + K)
    Xq = rng.integers(-127, 128, (M, K)).astype(np.int8)
    Wq, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=M, ids=(1,)))
    bias = synth.bias(N, seed=M, ids=(2,))
    packed, x, r = g.pack(dev(vals), dev(meta), K), dev(Xq), _rows(M)
    acc = oracle.spgemm_int8(Xq[r], vals, meta)
    assert np.array_equal(host(g.spgemm_int8(x, packed, N, out_dtype=torch.int32))[r], acc)
    s_a = np.float32(0.02)
    sa, sw, b = dev(np.array([s_a], np.float32)), dev(s_w), dev(bias)
    y = host(g.spgemm_int8(x, packed, N, act_scale=sa, w_scale=sw, bias=b))[r]
    assert np.array_equal(y.view(np.uint16), oracle.epilogue_int8_f32(acc, float(s_a), s_w, bias)["y16"].view(np.uint16))
    yg = host(g.spgemm_int8(x, packed, N, act_scale=sa, w_scale=sw, bias=b, gelu=True))[r]
    assert ulp_diff_f16(yg, oracle.epilogue_int8_f64(acc, float(s_a), s_w, bias, gelu=True)["y16"]).max() <= 1
    so = np.float32(np.abs(acc).max() * 0.02 * s_w.max() / 127.0)
    q = host(g.spgemm_int8(x, packed, N, act_scale=sa, w_scale=sw, out_dtype=torch.int8, out_scale=dev(np.array([so], np.float32))))[r]
    assert np.array_equal(q, oracle.epilogue_int8_f32(acc, float(s_a), s_w, None, out_scale=float(so))["q8"])


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_fp16(g, force_kernel, M, K, N):
    force_kernel(2)
    X, W, Wh, vals, meta, bias = fp16_problem(M, K, N, M)
    packed, x, r = g.pack(dev(vals), dev(meta), K), dev(X), _rows(M)
    _, a64 = oracle.spgemm_fp16(X[r], vals, meta)
    for gelu in (False, True):
        y = host(g.spgemm_fp16(x, packed, N, bias=dev(bias), gelu=gelu))[r]
        assert rel_err(y, oracle.epilogue_fp16_f64(a64, bias, gelu)["ref"]) <= 2e-3
