"""Flattened patches at the edges of the strip kernel: pieces of 1, 2, 4 and 8 bytes, rows of X of more 16-byte chunks than a
workgroup has threads, strips and planes that are not whole 16-byte vectors, and channels that do not fit into LDS together
(the kernel per channel)."""
import numpy as np
import pytest

from test_gpu_parity import dev, g, host  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# more than 256 strips, from which pieces of 1 and 2 bytes take the kernel that reads whole rows of patches: one and more than one batch
# of words in flight (2048 4-byte words, 1024 16-byte vectors), rows of X of more chunks than threads; and 256 strips
MANY = [(90, 3, 20, 40, 5, 80), (30, 3, 42, 308, 14, 592), (24, 11, 28, 224, 14, 2160), (130, 2, 28, 42, 14, 4112), (257, 1, 14, 42, 14, 208),
        (4, 1, 896, 28, 14, 208), (1, 257, 14, 28, 14, 50384), (1, 11, 28, 182, 14, 2160), (1, 12, 14, 112, 14, 2352)]


@pytest.mark.parametrize("B,C,H,W,P,K_pad", MANY + [(2, 3, 20, 40, 5, 80), (3, 1, 36, 12, 3, 16), (1, 2, 28, 42, 14, 4112), (2, 3, 42, 56, 14, 592),
                                             (1, 90, 28, 28, 14, 17648), (5, 3, 24, 40, 8, 208), (2, 3, 12, 20, 2, 16), (1, 3, 98, 14, 14, 640)])
@pytest.mark.parametrize("dtype", [np.float16, np.int8])
def test_patch_rows(g, B, C, H, W, P, K_pad, dtype):
    rng = np.random.default_rng(B * 1000 + W)
    img = rng.integers(-100, 100, (B, C, H, W)).astype(dtype)
    exp = np.zeros((B * (H // P) * (W // P), K_pad), dtype)
    exp[:, : C * P * P] = img.reshape(B, C, H // P, P, W // P, P).transpose(0, 2, 4, 1, 3, 5).reshape(-1, C * P * P)
    assert np.array_equal(host(g.im2col_patches(dev(img), P, K_pad)), exp)
