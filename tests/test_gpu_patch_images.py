"""The INT8 patch embedding with the quantiser of the images in one call (gpusq_patch_embed16_images), on the kernel that quantises whole rows
and on the others: codes and scale against the oracle's quantiser, tokens against its convolution's product."""
import numpy as np
import pytest

import oracle
from paper_2305_10727_amd import synth
from test_gpu_parity import dev, g, force_kernel, host, _oracle_weights  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _images(B, C, H, W, dtype, seed):
    return (np.random.default_rng(seed).standard_normal((B, C, H, W)) * 1.5).astype(dtype)


def _patches(codes):
    B, C, H, W = codes.shape
    return np.ascontiguousarray(codes.reshape(B, C, H // 16, 16, W // 16, 16).transpose(0, 2, 4, 1, 3, 5).reshape(B * (H // 16) * (W // 16), C * 256))


# one channel and three, rows of one patch and of odd numbers of them, chunks of patches of several images, one and two column blocks, several
# rounds; as the rules choose: the kernel for whole rows, the one for few rows, the tile kernel
@pytest.mark.parametrize("kernel,B,C,H,W,D", [(5, 40, 1, 112, 16, 1040), (5, 13, 3, 48, 208, 784), (5, 64, 3, 224, 224, 192), (5, 130, 3, 224, 240, 768), (-1, 64, 3, 224, 224, 768),
                                              (-1, 5, 3, 224, 224, 768), (-1, 64, 3, 224, 224, 1280), (-1, 300, 2, 64, 64, 256), (-1, 33, 3, 96, 160, 260)])
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
def test_images(g, force_kernel, kernel, B, C, H, W, D, dtype):
    force_kernel(kernel)
    img = _images(B, C, H, W, dtype, B + D)
    _, s_w, vals, meta = _oracle_weights(synth.weights(D, C * 256, seed=B, ids=(1,)))
    bias = synth.bias(D, seed=B, ids=(2,))
    exp_q, exp_s = oracle.quantize_tensor_int8(img.astype(np.float32).reshape(1, -1))
    X = _patches(exp_q.reshape(img.shape))
    M = len(X)
    r = np.unique(np.concatenate([np.arange(min(M, 300)), np.arange(max(0, M - 300), M), np.arange(0, M, 41)]))
    exp = oracle.epilogue_int8_f32(oracle.spgemm_int8(X[r], vals, meta), float(exp_s), s_w, bias)["y16"]
    Y, img_q = torch.full((M, D), 7.0, dtype=torch.float16, device="cuda"), torch.full((B, C, H, W), 99, dtype=torch.int8, device="cuda")
    sa, ws, x = torch.zeros(1, device="cuda"), torch.empty(4096, dtype=torch.uint8, device="cuda"), dev(img)
    g.calls.gpusq_patch_embed16_images(x, g._TORCH_DT[x.dtype], g.pack(dev(vals), dev(meta), C * 256), sa, dev(s_w), dev(bias), Y, img_q, ws, B, C, H, W, D, g.EPI_BIAS)
    assert host(sa)[0] == np.float32(exp_s) and np.array_equal(host(img_q).reshape(-1), exp_q.reshape(-1))
    assert np.array_equal(host(Y)[r].view(np.uint16), exp.view(np.uint16))


def _both(g, img, packed, sw, b, Y, ws, D):
    """(Y, codes, scale) of the one call into Y, and before it of the quantiser and the product apart"""
    B, C, H, W = img.shape
    q, s = g.quantize_int8(img.view(1, -1), g.PER_TENSOR)
    exp = torch.empty((B * (H // 16) * (W // 16), D), dtype=torch.float16, device="cuda")
    g.calls.gpusq_patch_embed16_int8(q, packed, s, sw, b, exp, B, C, H, W, D, g.EPI_BIAS)
    img_q, sa = torch.full((B, C, H, W), 99, dtype=torch.int8, device="cuda"), torch.full((1,), 1e3, device="cuda")
    g.calls.gpusq_patch_embed16_images(img, g._TORCH_DT[img.dtype], packed, sa, sw, b, Y, img_q, ws, B, C, H, W, D, g.EPI_BIAS)
    return (exp, q.view(-1), s), (Y, img_q.view(-1), sa)


# pixels that are no numbers, infinite, all zero, tiny; as the rules choose, the kernel for whole rows, the one for few rows, the tile kernel
@pytest.mark.parametrize("B,C,H,W,D", [(64, 3, 224, 224, 768), (5, 3, 224, 224, 768), (64, 3, 224, 224, 1536)])
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("kind", ["nan", "inf", "both", "zero", "tiny", "all nan"])
def test_pixels_that_leave_the_numbers(g, B, C, H, W, D, dtype, kind):
    img = (_images(B, C, H, W, np.float32, B) * {"zero": 0, "tiny": 1e-7}.get(kind, 1)).astype(dtype)
    for v, k in ((np.nan, ("nan", "both")), (np.inf, ("inf", "both")), (-np.inf, ("both",))):
        if kind in k: img.reshape(-1)[np.random.default_rng(len(k)).integers(0, img.size, 500)] = v
    if kind == "all nan": img[:] = np.nan
    _, s_w, vals, meta = _oracle_weights(synth.weights(D, C * 256, seed=B, ids=(1,)))
    Y, ws = torch.full((B * (H // 16) * (W // 16), D), 7.0, dtype=torch.float16, device="cuda"), torch.empty(4096, dtype=torch.uint8, device="cuda")
    exp, got = _both(g, dev(img), g.pack(dev(vals), dev(meta), C * 256), dev(s_w), dev(synth.bias(D, seed=B)), Y, ws, D)
    for e, t in zip(exp, got):
        assert np.array_equal(host(e), host(t), equal_nan=e.dtype != torch.int8)


# the tokens over the images, over their end and over the partial maxima of the range pass: as from buffers that lie apart
@pytest.mark.parametrize("how", ["images", "end", "workspace"])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_shared_operands(g, how, dtype):
    B, C, H, W, D = 64, 3, 224, 224, 768
    M, n = B * 196, B * C * H * W
    _, s_w, vals, meta = _oracle_weights(synth.weights(D, C * 256, seed=B, ids=(1,)))
    room = torch.empty(4 * n, dtype=torch.float16, device="cuda")
    img = room.view(dtype)[:n].view(B, C, H, W)
    img.copy_(dev(_images(B, C, H, W, np.float16, D)))
    at = {"images": 0, "end": n * img.element_size() // 2 - 768, "workspace": 2 * n}[how]
    Y = room[at:at + M * D].view(M, D)
    ws = Y.view(-1).view(torch.uint8)[:4096] if how == "workspace" else torch.empty(4096, dtype=torch.uint8, device="cuda")
    exp, got = _both(g, img, g.pack(dev(vals), dev(meta), C * 256), dev(s_w), dev(synth.bias(D, seed=B)), Y, ws, D)
    assert all(torch.equal(e, t) for e, t in zip(exp, got))


def test_refusals(g):
    B, C, H, W, D = 64, 3, 224, 224, 768
    img, Y = torch.zeros((B, C, H, W), dtype=torch.float16, device="cuda"), torch.empty((B * 196, D), dtype=torch.float16, device="cuda")
    q, sw, ws, sa = torch.full(img.shape, 99, dtype=torch.int8, device="cuda"), torch.ones(D, device="cuda"), torch.empty(4096, dtype=torch.uint8, device="cuda"), torch.zeros(1, device="cuda")
    packed = torch.zeros(g.packed_bytes(torch.int8, D, C * 256), dtype=torch.uint8, device="cuda")
    good = [img, g.F16, packed, sa, sw, None, Y, q, ws, B, C, H, W, D, 0]
    for at, value in ((1, g.I8), (3, None), (4, None), (7, None), (8, None), (11, 220), (14, g.EPI_GELU), (14, g.EPI_BIAS), (9, 1)):
        args = list(good)
        args[at] = value
        if at == 9:
            args[13] = 64  # too small for the gather: refused before the quantiser is launched
        with pytest.raises(g.GpusqError):
            g.calls.gpusq_patch_embed16_images(*args)
    torch.cuda.synchronize()
    assert (host(q) == 99).all()


# fewer than 2048 patches, by themselves on the kernel for whole rows (one channel: 256 values; 2^20 outputs) and not
@pytest.mark.parametrize("B,C,H,W,D", [(5, 1, 160, 192, 640), (1, 1, 336, 352, 576), (8, 3, 224, 224, 768), (5, 4, 240, 256, 900), (4, 3, 208, 176, 516)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_few_images_are_the_quantiser_and_the_product(g, B, C, H, W, D, dtype):
    r = torch.Generator(device="cuda").manual_seed(D)
    img = torch.randn((B, C, H, W), generator=r, device="cuda").to(dtype)
    w = g.prepare_weights(torch.randn((D, C * 256), generator=r, device="cuda") * 0.05, torch.int8)
    b, M = torch.randn(D, generator=r, device="cuda"), B * (H // 16) * (W // 16)
    q, s = g.quantize_int8(img.reshape(1, -1), g.PER_TENSOR)
    ref = g.patch_embed16(q.reshape(B, C, H, W), w["packed"], D, act_scale=s, w_scale=w["w_scale"], bias=b)
    Y, img_q, sa = torch.full((M, D), 7, dtype=torch.float16, device="cuda"), torch.full((B, C, H, W), 99, dtype=torch.int8, device="cuda"), torch.zeros(1, device="cuda")
    g.calls.gpusq_patch_embed16_images(img, g._TORCH_DT[dtype], w["packed"], sa, w["w_scale"], b, Y, img_q, torch.empty(4096, dtype=torch.uint8, device="cuda"), B, C, H, W, D, g.EPI_BIAS)
    assert torch.equal(img_q.reshape(-1), q.reshape(-1)) and torch.equal(sa, s.reshape(1)) and torch.equal(Y.view(torch.int16), ref.view(torch.int16))
