"""K that is no whole number of 128-byte steps on the tile kernel with one workgroup per CU: every size of the last step's tail, one
step to a tile and more, several rounds of tiles, widths that are no whole lines; infinities and NaN in the last step."""
import numpy as np
import pytest

import oracle
from paper_2305_10727_amd import synth
from test_gpu_parity import dev, fp16_problem, g, force_kernel, host, rel_err, _oracle_weights  # noqa: F401
from test_gpu_tile_heights import _rows

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(3067, 16, 1024), (1020, 48, 520), (5000, 144, 520), (3000, 592, 1280), (20000, 208, 1024), (6000, 336, 300), (12608, 576, 768), (700, 1008, 520), (900, 96, 4)]


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_int8(g, force_kernel, M, K, N):
    force_kernel(2)
    Xq = np.random.default_rng(M + K).integers(-127, 128, (M, K)).astype(np.int8)
    Wq, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=M, ids=(1,)))
    bias = synth.bias(N, seed=M, ids=(2,))
    packed, x, r = g.pack(dev(vals), dev(meta), K), dev(Xq), _rows(M)
    acc = oracle.spgemm_int8(Xq[r], vals, meta)
    assert np.array_equal(host(g.spgemm_int8(x, packed, N, out_dtype=torch.int32))[r], acc)
    s_a = np.float32(0.02)
    y = host(g.spgemm_int8(x, packed, N, act_scale=dev(np.array([s_a], np.float32)), w_scale=dev(s_w), bias=dev(bias)))[r]
    assert np.array_equal(y.view(np.uint16), oracle.epilogue_int8_f32(acc, float(s_a), s_w, bias)["y16"].view(np.uint16))


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_fp16(g, force_kernel, M, K, N):
    force_kernel(2)
    X, W, Wh, vals, meta, bias = fp16_problem(M, K, N, M)
    packed, r = g.pack(dev(vals), dev(meta), K), _rows(M)
    _, a64 = oracle.spgemm_fp16(X[r], vals, meta)
    y = host(g.spgemm_fp16(dev(X), packed, N, bias=dev(bias)))[r]
    assert rel_err(y, oracle.epilogue_fp16_f64(a64, bias, False)["ref"]) <= 2e-3
    # an infinity or a NaN reaches the outputs whose weights keep its column and no others, as on the small kernel
    X[::3, -(K % 64 or 64)] = np.inf
    X[1::7, -1] = np.nan
    y = g.spgemm_fp16(dev(X), packed, N)
    force_kernel(1)
    ref = g.spgemm_fp16(dev(X), packed, N)
    assert torch.equal(torch.isfinite(y), torch.isfinite(ref)) and torch.equal(torch.isnan(y), torch.isnan(ref))


def test_fp16_input_of_the_int8_product(g):
    """Many rows take the tile kernel; the product that quantises its input keeps the small kernels for every ragged K."""
    M, K, N = 12544, 592, 1280
    assert g.spgemm_plan(torch.int8, M, N, K)["kernel"] == 2 and g.spgemm_plan(torch.float16, M, N, K)["kernel"] == 2
    Wq, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=3, ids=(1,)))
    packed = g.pack(dev(vals), dev(meta), K)
    X = torch.randn((M, K), device="cuda").half()
    Xq, s = g.quantize_int8(X, g.PER_TENSOR)
    a = g.spgemm_int8_xf16(X, packed, N, s, dev(s_w), out_dtype=torch.int32)
    assert torch.equal(a, g.spgemm_int8(Xq, packed, N, out_dtype=torch.int32))


# both sides of the lines between the 64 x 64 tiles, the 128 x 128 tiles and tile kernel 2 (and of the kernel for few rows where fp16 is
# quantised on the way in): each output type as from the 64 x 64 tiles
@pytest.mark.parametrize("M,K,N", [(3136, 192, 640), (3137, 192, 704), (8192, 192, 1024), (8193, 192, 1024), (6304, 272, 576), (25216, 64, 128),
                                   (8192, 64, 64), (8193, 64, 64), (16400, 64, 64)])
def test_choice_by_size(g, force_kernel, M, K, N):
    Wq, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=N, ids=(3,)))
    packed, sw, bias = g.pack(dev(vals), dev(meta), K), dev(s_w), dev(synth.bias(N, seed=M, ids=(4,)))
    X = torch.randn((M, K), generator=torch.Generator(device="cuda").manual_seed(M), device="cuda").half()
    Xq, s = g.quantize_int8(X, g.PER_TENSOR)
    so = dev(np.array([0.05], np.float32))
    outs = lambda x, f: [f(x, packed, N, s, sw, bias, out_dtype=dt, out_scale=so if dt == torch.int8 else None) for dt in (torch.float16, torch.int8, torch.int32)]
    own, xf16 = outs(Xq, g.spgemm_int8), outs(X, g.spgemm_int8_xf16)
    w16 = g.prepare_weights(dev(synth.weights(N, K, seed=N, ids=(5,))), torch.float16)["packed"]
    y16 = g.spgemm_fp16(X, w16, N, bias)
    force_kernel(0)
    for a, b, c in zip(own, xf16, outs(Xq, g.spgemm_int8)):
        assert torch.equal(a, c) and torch.equal(b, c)
    assert rel_err(host(y16), host(g.spgemm_fp16(X, w16, N, bias))) <= 2e-3
