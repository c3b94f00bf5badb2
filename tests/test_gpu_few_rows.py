"""The sparse GEMM's kernel for few rows (K steps dealt out over the wavefronts of a workgroup, 64-channel x 16- or 32-row
tiles) and the one-call INT8 layer built on it, against the CPU oracle: sizes at the edges of its tiles, K steps fewer than
wavefronts, one more than a batch of steps, and a K that ends inside a step."""
import numpy as np
import pytest

import oracle
from paper_2305_10727_amd import synth
from test_gpu_parity import FP16_SHAPES, dev, fp16_problem, g, force_kernel, host, rel_err, ulp_diff_f16, _oracle_weights  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# M: one row, one tile of 16 or 32 rows and one row more, several; N: one group of 4, one 64-channel block and 4 more, 1000
# classes, enough blocks for the 32-row tiles; K: a single chunk, less and more than 4 steps, a ragged last step, more than
# 12 steps (8 wavefronts) and more than 24 (a second batch)
SHAPES = [(1, 16, 4, 1), (16, 128, 64, 2), (17, 144, 68, 3), (33, 640, 132, 4), (64, 768, 1000, 5), (197, 768, 2304, 6),
          (333, 1040, 520, 7), (31, 1680, 260, 8), (50, 3344, 100, 9), (600, 384, 1536, 10)]


@pytest.mark.parametrize("M,K,N,seed", SHAPES)
def test_int8_accumulators_and_epilogues(g, force_kernel, M, K, N, seed):
    force_kernel(4)
    rng = np.random.default_rng(seed)
    Xq = rng.integers(-127, 128, (M, K)).astype(np.int8)
    Wq, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=seed, ids=(1,)))
    bias = synth.bias(N, seed=seed, ids=(2,))
    packed = g.pack(dev(vals), dev(meta), K)
    acc = oracle.spgemm_int8(Xq, vals, meta)
    assert np.array_equal(host(g.spgemm_int8(dev(Xq), packed, N, out_dtype=torch.int32)), acc)
    s_a, so = np.float32(0.02), np.float32(max(np.abs(acc).max(), 1) * 0.02 * s_w.max() / 127.0)
    sa, sw, b = dev(np.array([s_a], np.float32)), dev(s_w), dev(bias)
    y = host(g.spgemm_int8(dev(Xq), packed, N, act_scale=sa, w_scale=sw, bias=b))
    assert np.array_equal(y.view(np.uint16), oracle.epilogue_int8_f32(acc, float(s_a), s_w, bias)["y16"].view(np.uint16))
    yg = host(g.spgemm_int8(dev(Xq), packed, N, act_scale=sa, w_scale=sw, bias=b, gelu=True))
    assert ulp_diff_f16(yg, oracle.epilogue_int8_f64(acc, float(s_a), s_w, bias, gelu=True)["y16"]).max() <= 1
    q = host(g.spgemm_int8(dev(Xq), packed, N, act_scale=sa, w_scale=sw, out_dtype=torch.int8, out_scale=dev(np.array([so], np.float32))))
    assert np.array_equal(q, oracle.epilogue_int8_f32(acc, float(s_a), s_w, None, out_scale=float(so))["q8"])


@pytest.mark.parametrize("M,K,N,seed", SHAPES)
def test_fp16(g, force_kernel, M, K, N, seed):
    force_kernel(4)
    X, W, Wh, vals, meta, bias = fp16_problem(M, K, N, seed)
    packed = g.pack(dev(vals), dev(meta), K)
    _, a64 = oracle.spgemm_fp16(X, vals, meta)
    for gelu in (False, True):
        y = host(g.spgemm_fp16(dev(X), packed, N, bias=dev(bias), gelu=gelu))
        assert rel_err(y, oracle.epilogue_fp16_f64(a64, bias, gelu)["ref"]) <= 2e-3


def _layer(g, X, packed, sw, b, M, N, K, scale=None, gelu=False):
    """gpusq_linear_int8 on X [M, K]: (Y, codes, scale)"""
    from paper_2305_10727_amd.pipeline import _p
    Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    Xq = torch.full((M, K), 99, dtype=torch.int8, device="cuda")
    sa = torch.empty(1, dtype=torch.float32, device="cuda") if scale is None else scale
    ws = torch.empty(4096, dtype=torch.uint8, device="cuda")
    st = g.lib().gpusq_linear_int8(_p(X), g._TORCH_DT[X.dtype], _p(packed), _p(sa), int(scale is not None), _p(sw), _p(b), _p(Y), g.F16, None,
                                   _p(Xq), _p(ws), M, N, K, g._epi(b, gelu), g._stream())
    assert st == g.OK
    return host(Y), host(Xq), host(sa)


# the range of X found by every workgroup (small X) and by a pass of its own, the codes written by the first column of tiles,
# fp32 activations and a problem of the tile kernels (quantiser and GEMM one behind the other); 8 wavefronts for a long range
# (331 x 192) and for one workgroup of many steps, several batches of them per wavefront
@pytest.mark.parametrize("M,K,N,seed", SHAPES + [(700, 768, 512, 11), (4100, 256, 384, 12), (331, 192, 384, 13), (16, 1536, 64, 14), (20, 5120, 196, 15), (40, 3088, 64, 16)])
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("given", [False, True])
def test_one_call_layer(g, M, K, N, seed, dtype, given):
    rng = np.random.default_rng(seed + 100)
    X = (rng.standard_normal((M, K)) * 1.5).astype(dtype)
    if given:
        X.reshape(-1)[:8] = np.array([0.0, -0.0, 65504.0, -65504.0, 6e-8, np.inf, -np.inf, np.nan], dtype)  # clamped, 0
    Wq, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=seed, ids=(3,), sigma=0.05))
    bias = synth.bias(N, seed=seed, ids=(4,))
    packed, sw, b = g.pack(dev(vals), dev(meta), K), dev(s_w), dev(bias)
    scale = np.float32(4.0 / 127.0) if given else None
    exp_q, exp_s = oracle.quantize_tensor_int8(X.astype(np.float32), scale=None if scale is None else float(scale))
    acc = oracle.spgemm_int8(exp_q, vals, meta)
    y, q, s = _layer(g, dev(X), packed, sw, b, M, N, K, None if scale is None else dev(np.array([scale])))
    assert s[0] == np.float32(exp_s) and np.array_equal(q, exp_q)
    assert np.array_equal(y.view(np.uint16), oracle.epilogue_int8_f32(acc, float(s[0]), s_w, bias)["y16"].view(np.uint16))


def test_fp16_codes_decide_as_the_division_does(g):
    """Every finite fp16 value under many scales, those included for which values lie on a code boundary (so that the
    single fused multiply-add would decide wrongly), denormal, huge and zero scales: the codes are rint(x / s) with the
    IEEE division, clamped."""
    h = np.arange(0, 0x7C00, dtype=np.uint16).view(np.float16)
    X = np.concatenate([h, -h]).reshape(62, 1024)
    N, K = 4, 1024
    Wq, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=1))
    packed, sw, b = g.pack(dev(vals), dev(meta), K), dev(s_w), dev(synth.bias(N))
    rng = np.random.default_rng(3)
    scales = [np.float32(v) for v in (1.0, 0.1, 1 / 3, 2 / 3, 0.7, 1e-3, 3e-5, 5e-8, 511.5, 65504 / 127, 1e-38, 1e-45, 1e38, 0.0, np.inf)]
    scales += list(rng.uniform(0.01, 1.0, 12).astype(np.float32))
    # fp16 values divided by half-integers: on the boundary, or one rounding away from it
    scales += [np.float32(np.float32(v) / np.float32(c + 0.5)) for v, c in zip(rng.uniform(0.5, 2.0, 40).astype(np.float16), rng.integers(0, 127, 40))]
    for s in scales:
        with np.errstate(all="ignore"):
            exp, _ = oracle.quantize_tensor_int8(X.astype(np.float32), scale=float(s))
        _, q, _ = _layer(g, dev(X), packed, sw, b, 62, N, K, dev(np.array([s], np.float32)))
        assert np.array_equal(q, exp), s


def test_codes_under_scales_one_unit_off_a_power_of_two(g):
    """One unit below a power of two a rounded reciprocal and one correction do not give the rounded quotient of half the scale, which
    lies on the boundary between codes 0 and 1: the codes are those of the division there, given and found."""
    X = np.arange(0, 0x7C00, 7, dtype=np.uint16)[:2048].view(np.float16).reshape(2, 1024)
    N, K = 4, 1024
    _, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=1))
    packed, sw, b = g.pack(dev(vals), dev(meta), K), dev(s_w), dev(synth.bias(N))
    for e in range(-8, 9):
        p = np.float32(2.0 ** e)
        for s in (np.nextafter(p, np.float32(0)), p, np.nextafter(p, np.float32(1e9))):
            x = X.copy()
            x[0, :4] = np.array([p / 2, -p / 2, 1.5 * p, -2.5 * p], np.float16)
            exp, _ = oracle.quantize_tensor_int8(x.astype(np.float32), scale=float(s))
            assert np.array_equal(_layer(g, dev(x), packed, sw, b, 2, N, K, dev(np.array([s])))[1], exp), s


# fp32 activations quantised by the kernel for few rows: 4 and 8 wavefronts, one and two workgroups per CU, the range found by every
# workgroup and by a pass, rows that end inside a K step; NaN and infinities beside a given scale; int8 output
@pytest.mark.parametrize("M,K,N", [(1, 16, 4), (50, 192, 260), (331, 192, 384), (700, 384, 512), (33, 656, 132), (197, 1536, 64), (17, 1040, 68)])
@pytest.mark.parametrize("given", [False, True])
def test_one_call_layer_of_fp32_rows(g, M, K, N, given):
    assert g.lib().gpusq_linear_int8_launches(g.F32, M, N, K, g.EPI_BIAS, int(given), 0) < (2 if given else 3)
    rng = np.random.default_rng(M + K)
    X = (rng.standard_normal((M, K)) * 1.5).astype(np.float32)
    if given:
        X.reshape(-1)[:8] = np.array([0.0, -0.0, 3e38, -3e38, 1e-40, np.inf, -np.inf, np.nan], np.float32)
    _, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=M, ids=(9,), sigma=0.05))
    bias = synth.bias(N, seed=M, ids=(10,))
    packed, sw, b = g.pack(dev(vals), dev(meta), K), dev(s_w), dev(bias)
    scale = np.float32(4.0 / 127.0) if given else None
    exp_q, exp_s = oracle.quantize_tensor_int8(X, scale=None if scale is None else float(scale))
    acc = oracle.spgemm_int8(exp_q, vals, meta)
    y, q, s = _layer(g, dev(X), packed, sw, b, M, N, K, None if scale is None else dev(np.array([scale])))
    assert s[0] == np.float32(exp_s) and np.array_equal(q, exp_q)
    assert np.array_equal(y.view(np.uint16), oracle.epilogue_int8_f32(acc, float(s[0]), s_w, bias)["y16"].view(np.uint16))
    so = np.float32(np.abs(acc).max() * s[0] * s_w.max() / 127.0 + 1e-9)
    Y, Xq, sa = torch.empty((M, N), dtype=torch.int8, device="cuda"), torch.empty((M, K), dtype=torch.int8, device="cuda"), dev(s.copy())
    g.calls.gpusq_linear_int8(dev(X), g.F32, packed, sa, int(given), sw, b, Y, g.I8, dev(np.array([so])), Xq, torch.empty(4096, dtype=torch.uint8, device="cuda"), M, N, K, g.EPI_BIAS)
    assert np.array_equal(host(Y), oracle.epilogue_int8_f32(acc, float(s[0]), s_w, bias, out_scale=float(so))["q8"])


# a square layer run on its own output, whole or partly over X, or from half of the bytes of fp32 rows on (right behind fp16 ones): as
# from a copy of X, where the GEMM would quantise for itself
@pytest.mark.parametrize("M,K", [(64, 768), (197, 768), (16, 256)])
@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("shift", [0, 8, -8, "M * K"])
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
def test_one_call_layer_writes_over_its_input(g, M, K, given, shift, dtype):
    N, shift, x_dt = K, M * K if shift == "M * K" else shift, g.F16 if dtype == np.float16 else g.F32
    assert g.lib().gpusq_linear_int8_launches(x_dt, M, N, K, g.EPI_BIAS, int(given), 0) < (2 if given else 3)
    Wq, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=M, ids=(5,), sigma=0.05))
    packed, sw, b = g.pack(dev(vals), dev(meta), K), dev(s_w), dev(synth.bias(N, seed=M, ids=(6,)))
    X = (np.random.default_rng(M).standard_normal((M, K)) * 1.5).astype(dtype)
    scale = dev(np.array([4 / 127], np.float32)) if given else torch.empty(1, dtype=torch.float32, device="cuda")
    y, q, s = _layer(g, dev(X), packed, sw, b, M, N, K, scale if given else None)
    buf = torch.zeros(3 * M * K + 16, dtype=torch.float16, device="cuda")
    x, over = buf[8:8 + M * K * X.itemsize // 2].view(dev(X).dtype), buf[8 + shift:8 + shift + M * N]
    x.copy_(dev(X).view(-1))
    Xq, ws = torch.full((M, K), 99, dtype=torch.int8, device="cuda"), torch.empty(4096, dtype=torch.uint8, device="cuda")
    g.calls.gpusq_linear_int8(x, x_dt, packed, scale, int(given), sw, b, over, g.F16, None, Xq, ws, M, N, K, g.EPI_BIAS)
    assert np.array_equal(host(Xq), q) and host(scale)[0] == s[0]
    assert np.array_equal(host(over).reshape(M, N).view(np.uint16), y.view(np.uint16))


# out_scale the activation scale that the call itself finds (by every workgroup, or behind a range pass), and Y over the partial
# maxima of the range pass: as from operands that lie apart
@pytest.mark.parametrize("M,K,N,dtype", [(64, 768, 1000, np.float16), (197, 768, 768, np.float16), (197, 768, 2304, np.float16), (64, 768, 1000, np.float32),
                                         (197, 768, 768, np.float32), (197, 512, 2304, np.float32), (40, 256, 512, np.float32)])
@pytest.mark.parametrize("out", ["scale", "workspace"])
def test_one_call_layer_with_shared_operands(g, M, K, N, dtype, out):
    x_dt = g.F16 if dtype == np.float16 else g.F32
    assert g.lib().gpusq_linear_int8_launches(x_dt, M, N, K, g.EPI_BIAS, 0, 0) < 3
    Wq, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=M, ids=(7,), sigma=0.05))
    packed, sw, b = g.pack(dev(vals), dev(meta), K), dev(s_w), dev(synth.bias(N, seed=M, ids=(8,)))
    x = dev((np.random.default_rng(N).standard_normal((M, K)) * 1.5).astype(dtype))
    exp_q, exp_s = g.quantize_int8(x, g.PER_TENSOR)
    Xq, scale = torch.empty((M, K), dtype=torch.int8, device="cuda"), torch.full((1,), 1e3, device="cuda")
    if out == "scale":  # the scale in memory before the call is another one
        Y, ws = torch.empty((M, N), dtype=torch.int8, device="cuda"), torch.empty(4096, dtype=torch.uint8, device="cuda")
        exp = g.spgemm_int8(exp_q, packed, N, act_scale=exp_s, w_scale=sw, bias=b, out_dtype=torch.int8, out_scale=exp_s)
        g.calls.gpusq_linear_int8(x, x_dt, packed, scale, 0, sw, b, Y, g.I8, scale, Xq, ws, M, N, K, g.EPI_BIAS)
    else:
        Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
        exp = g.spgemm_int8(exp_q, packed, N, act_scale=exp_s, w_scale=sw, bias=b)
        g.calls.gpusq_linear_int8(x, x_dt, packed, scale, 0, sw, b, Y, g.F16, None, Xq, Y, M, N, K, g.EPI_BIAS)
    assert torch.equal(Xq, exp_q) and torch.equal(scale, exp_s) and torch.equal(Y, exp)


# as many rows as the kernel for whole rows asks for, of so few channels that the kernel for few rows takes them: with and without the codes
@pytest.mark.parametrize("M,K,N", [(2048, 256, 64), (4096, 256, 64), (8192, 256, 64)])
def test_many_rows_of_one_block(g, M, K, N):
    from paper_2305_10727_amd.pipeline import SparseLinear
    lin = SparseLinear(M, K, N, "int8")
    assert lin.takes_fp16_input()
    lin.prepare_weights(dev(synth.weights(N, K, seed=M)))
    x, b = dev((np.random.default_rng(M).standard_normal((M, K)) * 1.5).astype(np.float16)), dev(synth.bias(N, seed=M))
    lin.act_scale.fill_(4 / 127)
    exp_q, _ = g.quantize_int8(x, g.PER_TENSOR, scale=lin.act_scale)
    exp = g.spgemm_int8(exp_q, lin.packed, N, act_scale=lin.act_scale, w_scale=lin.w_scale, bias=b)
    lin.Xq.fill_(99)
    assert torch.equal(lin.gemm_from_f16(x, b), exp) and (lin.Xq == 99).all()
    lin.Y.zero_()
    assert torch.equal(lin.forward(x, b, static=True), exp) and torch.equal(lin.Xq, exp_q)
