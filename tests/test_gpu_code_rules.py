"""The codes of the activation and weight quantisers where the definition, clamp(rint(x / s)) with the IEEE fp32 division and 0 for
NaN, leaves no room: every fp16 value under given scales, infinities and NaN included, through each entry point that makes codes of
fp16 activations, element by element against the CPU oracle."""
import numpy as np
import pytest

import oracle
from test_gpu_few_rows import _layer, _oracle_weights
from test_gpu_parity import dev, g, force_kernel, host  # noqa: F401
from paper_2305_10727_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

M, K = 64, 1024


def _every_fp16():
    """[64, 1024] matrices: every fp16 value but NaN, each infinity the only one of its wavefront; the same with a NaN in every
    vector of 8, at two places so that every value is met; infinities of both signs and NaN in every vector."""
    h = np.arange(0, 0x7C01, dtype=np.uint16).view(np.float16)
    plain = np.resize(np.concatenate([h, -h]), (M, K))
    with_nan = []
    for at in (2, 7):
        x = plain.copy()
        x[:, at::8] = np.nan
        with_nan.append(x)
    mixed = plain.copy()
    mixed[:, 0::8], mixed[:, 3::8], mixed[::2, 6::8] = np.inf, -np.inf, np.nan
    return [plain, *with_nan, mixed]


def _codes_of_every_entry_point(g, force_kernel, X, s):
    """(name, codes [64, 1024]) of X under the given scale"""
    x, scale = dev(X), dev(np.array([s], np.float32))
    yield "quantize_int8", host(g.quantize_int8(x, g.PER_TENSOR, scale=scale)[0])
    xq = torch.full((M, K), 99, dtype=torch.int8, device="cuda")
    yield "quantize_tensor_int8_noalloc", host(g.quantize_tensor_int8_noalloc(x, xq, scale, scale_is_input=True)[0])
    N = 4
    _, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=1))
    yield "linear_int8", _layer(g, x, g.pack(dev(vals), dev(meta), K), dev(s_w), dev(synth.bias(N)), M, N, K, scale)[1]
    # the product with the unit matrix: accumulators that are the codes
    packed = g.pack(*g.compress(torch.eye(K, dtype=torch.int8, device="cuda")), K)
    for kernel in (4, 0):
        force_kernel(kernel)
        y = g.spgemm_int8_xf16(x, packed, K, scale, torch.ones(K, device="cuda"), out_dtype=torch.int32)
        yield "spgemm_int8_xf16, kernel %d" % kernel, host(y)


# scales under which values lie on code boundaries, so that the quantiser refines its products (0.03 ... 3/64), and others;
# negative scales decide as the division does too
@pytest.mark.parametrize("s", [0.03, 0.07, 0.7, 0.75, 3 / 64, 4 / 127, 1.0, 0.1, -0.03, -0.75, -3 / 64, -4 / 127])
def test_given_scale(g, force_kernel, s):
    for X in _every_fp16():
        exp, _ = oracle.quantize_tensor_int8(X.astype(np.float32), scale=float(np.float32(s)))
        for name, q in _codes_of_every_entry_point(g, force_kernel, X, s):
            assert np.array_equal(q, exp), name
