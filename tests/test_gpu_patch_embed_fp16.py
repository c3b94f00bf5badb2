"""Patch embeddings from fp16 images in one launch (gpusq_patch_embed_fp16) against the oracle's convolution and against the two calls that it stands for."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import dev, force_kernel, g, host  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _weights(g, C, P, D, K_pad, seed):
    W = np.zeros((D, K_pad), np.float32)
    W[:, : C * P * P] = np.random.default_rng(seed).normal(size=(D, C * P * P)).astype(np.float32) * 0.1
    W = oracle.prune_2to4(W)[0]
    return W, g.prepare_weights(dev(W), torch.float16)["packed"]


def _call(g, img, packed, bias, K_pad, P, D, Y=None):
    B, C, H, W = img.shape
    M = B * (H // P) * (W // P)
    X = torch.full((M, K_pad), 7, dtype=torch.float16, device="cuda")
    Y = torch.full((M, D), 7, dtype=torch.float16, device="cuda") if Y is None else Y
    g.calls.gpusq_patch_embed_fp16(img, packed, bias, Y, X, B, C, H, W, P, K_pad, D, 0 if bias is None else g.EPI_BIAS)
    return Y, X


# a patch; part of a slab and of an image row's patches; 1 to 4 slabs to a workgroup, the last part of one; rows of 2 to 28 pixels, fewer and more than the rows in
# flight; one K step to 20, whole and not; one block of channels, as many as wavefronts, one more; K_pad beyond the last step's; a second round of workgroups
SIZES = [(1, 3, 14, 14, 14, 592, 64), (2, 3, 42, 70, 14, 592, 320), (9, 3, 224, 224, 14, 640, 256), (1, 1, 6, 10, 2, 16, 64), (3, 3, 24, 40, 4, 48, 192),
         (5, 3, 64, 72, 8, 192, 128), (2, 1, 84, 56, 28, 784, 64), (40, 3, 224, 224, 14, 592, 64), (50, 3, 224, 224, 14, 592, 64), (130, 3, 224, 224, 14, 592, 128),
         (3, 5, 60, 84, 12, 768, 64), (2, 6, 42, 28, 14, 1184, 64), (2, 3, 42, 28, 14, 720, 64), (1, 2, 64, 96, 32, 2048, 64)]


@pytest.mark.parametrize("B,C,H,W,P,K_pad,D", SIZES)
def test_one_launch_matches_the_oracle_and_the_two(g, force_kernel, B, C, H, W, P, K_pad, D):
    rng = np.random.default_rng(B + H)
    img = rng.normal(size=(B, C, H, W)).astype(np.float16)
    K = C * P * P
    wt, packed = _weights(g, C, P, D, K_pad, 3)
    bias = dev(rng.normal(size=D).astype(np.float32))
    force_kernel(6)
    assert g.lib().gpusq_patch_embed_fp16_launches(B, C, H, W, P, K_pad, D, g.EPI_BIAS, 0) == 1
    Y, X = _call(g, dev(img), packed, bias, K_pad, P, D)
    plain, _ = _call(g, dev(img), packed, None, K_pad, P, D)
    assert bool((X == 7).all())  # (left as it is)
    force_kernel(None)
    two = g.spgemm_fp16(g.im2col_patches(dev(img), P, K_pad), packed, D, bias=bias)
    # sums of K products of values of 1 and 0.1 in another order
    assert torch.allclose(Y.float(), two.float(), rtol=2e-3, atol=2e-3)
    n = min(B, 2)
    a64, _ = oracle.patch_conv_f16(img[:n], wt.astype(np.float16)[:, :K].reshape(D, C, P, P))
    expected = a64.reshape(-1, D)
    rows = expected.shape[0]
    tol = 2.0 ** -10 * np.abs(expected) + 2.0 ** -20 * K  # half a unit of the fp16 result twice over, and the fp32 sums
    assert (np.abs(host(plain)[:rows].astype(np.float64) - expected) <= tol).all()
    assert (np.abs(host(Y)[:rows].astype(np.float64) - (expected + host(bias)[None].astype(np.float64))) <= tol + 2.0 ** -10 * np.abs(host(bias))[None]).all()


# two slabs to a workgroup (on 256 CUs): 320 slabs of patches; 307 of them where LDS holds no more, the last workgroup with four patches
@pytest.mark.parametrize("B,C,H,W,P,K_pad,D", [(20, 3, 224, 224, 14, 592, 64), (25, 3, 252, 252, 18, 976, 64)])
def test_two_slabs(g, force_kernel, B, C, H, W, P, K_pad, D):
    test_one_launch_matches_the_oracle_and_the_two(g, force_kernel, B, C, H, W, P, K_pad, D)


@pytest.mark.parametrize("W", [14, 98, 126, 210, 224])  # (tails of patches in the last workgroup)
def test_every_patch_and_pixel_is_met_once(g, force_kernel, W):
    """Weights that pick single pixels: Y holds the images, bit for bit"""
    B, C, H, P, K_pad, D = 3, 3, 42, 14, 592, 640
    img = np.random.default_rng(W).normal(size=(B, C, H, W)).astype(np.float16)
    wt = np.zeros((D, K_pad), np.float32)
    wt[np.arange(C * P * P), np.arange(C * P * P)] = 1
    packed = g.prepare_weights(dev(wt), torch.float16)["packed"]
    force_kernel(6)
    Y, _ = _call(g, dev(img), packed, None, K_pad, P, D)
    force_kernel(None)
    X = g.im2col_patches(dev(img), P, K_pad)
    assert torch.equal(Y[:, : C * P * P], X[:, : C * P * P])
    assert not bool(Y[:, C * P * P:].any())


def test_images_under_the_output_are_two_launches(g, force_kernel):
    B, C, H, W, P, K_pad, D = 8, 3, 28, 28, 14, 592, 64
    img = dev(np.random.default_rng(1).normal(size=(B, C, H, W)).astype(np.float16))
    _, packed = _weights(g, C, P, D, K_pad, 5)
    force_kernel(6)
    expected, _ = _call(g, img, packed, None, K_pad, P, D)
    Y = img.view(-1)[: expected.numel()].view(expected.shape)
    got, X = _call(g, img, packed, None, K_pad, P, D, Y=Y)
    assert not bool((X == 7).all())
    assert torch.allclose(got.float(), expected.float(), rtol=2e-3, atol=2e-3)


def test_not_a_number_and_infinities_reach_their_own_patches_only(g, force_kernel):
    B, C, H, W, P, K_pad, D = 2, 3, 56, 56, 14, 640, 64
    img = np.random.default_rng(2).normal(size=(B, C, H, W)).astype(np.float16)
    img[0, 1, 3, 17] = np.nan
    img[1, 2, 55, 55] = np.inf
    _, packed = _weights(g, C, P, D, K_pad, 7)
    force_kernel(6)
    Y = host(_call(g, dev(img), packed, None, K_pad, P, D)[0]).reshape(B, 4, 4, D)
    finite = np.isfinite(Y).all(axis=3)
    assert not np.isfinite(Y[0, 0, 1]).all() and not np.isfinite(Y[1, 3, 3]).all()
    finite[0, 0, 1] = finite[1, 3, 3] = True
    assert finite.all()


def test_patch_embed_of_the_pipeline_in_a_graph(g):
    """SparsePatchEmbed, fp16: one call, the same under capture on every replay"""
    from paper_2305_10727_amd.pipeline import SparsePatchEmbed
    B, C, H, W, P, D = 9, 3, 224, 224, 14, 192
    r = torch.Generator(device="cuda").manual_seed(1)
    wt = torch.randn((D, C, P, P), generator=r, device="cuda") * 0.05
    bias = torch.randn(D, generator=r, device="cuda")
    e, apart = SparsePatchEmbed(B, C, H, W, P, D, "fp16"), SparsePatchEmbed(B, C, H, W, P, D, "fp16", fused=False)
    assert e.one_call and not apart.one_call and not apart.fused
    assert g.lib().gpusq_patch_embed_fp16_launches(B, C, H, W, P, e.K_pad, D, e.linear.epilogue, 0) == 1
    e.prepare_weights(wt)
    apart.prepare_weights(wt)
    img = torch.empty((B, C, H, W), dtype=torch.float16, device="cuda")
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    img.normal_(generator=r)
    with torch.cuda.stream(s):
        e.forward(img, bias)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=s):
        y = e.forward(img, bias)
    for _ in range(3):
        img.normal_(generator=r)
        graph.replay()
        torch.cuda.synchronize()
        replayed = y.clone()
        assert torch.equal(replayed, e.forward(img, bias))
        assert torch.allclose(replayed.float(), apart.forward(img, bias).float(), rtol=2e-3, atol=2e-3)
