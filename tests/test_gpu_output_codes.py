"""fp16 output and its codes in one launch (gpusq_spgemm_int8_codes) on every kernel that has such an epilogue, against the CPU
oracle: output, then quantiser, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2305_10727_amd import synth
from test_gpu_parity import dev, g, force_kernel, host, _oracle_weights  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# the kernel for few rows (one row, one more than a tile, N of 4 more than a block), the small kernels' tiles and one row more, the tile
# kernel: whole lines, a last tile partly outside Y in both directions, N of no whole 16 (half and whole pieces), a ragged K, several rounds;
# kernel 3 where it is asked for (the tile kernel runs); as the rules choose
@pytest.mark.parametrize("kernel,M,K,N", [(4, 1, 16, 4), (4, 33, 768, 132), (4, 197, 640, 768), (0, 65, 192, 68), (0, 300, 768, 256), (1, 129, 128, 132), (1, 400, 144, 256),
                                          (2, 2048, 384, 768), (2, 1111, 512, 272), (2, 1111, 512, 264), (2, 700, 256, 260), (2, 3000, 272, 528), (2, 20011, 128, 1040),
                                          (3, 2100, 256, 512), (-1, 12544, 512, 512), (-1, 1576, 384, 384)])
@pytest.mark.parametrize("biased", [False, True])
def test_output_and_codes(g, force_kernel, kernel, M, K, N, biased):
    force_kernel(kernel)
    rng = np.random.default_rng(M + N)
    Xq = rng.integers(-127, 128, (M, K)).astype(np.int8)
    _, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=M, ids=(1,)))
    bias = synth.bias(N, seed=M, ids=(2,)) if biased else None
    rows = np.unique(np.concatenate([np.arange(min(M, 80)), np.arange(max(0, M - 80), M), rng.integers(0, M, 100)]))
    acc = oracle.spgemm_int8(Xq[rows], vals, meta)
    s_a = np.float32(0.02)
    y = oracle.epilogue_int8_f32(acc, float(s_a), s_w, bias)["y16"]
    # a scale that the largest outputs exceed
    s_y = np.float32(np.abs(y.astype(np.float32)).max() / 100.0 + 1e-9)
    codes, _ = oracle.quantize_tensor_int8(y.astype(np.float32), scale=float(s_y))
    Y, Yq = torch.full((M, N), 7.0, dtype=torch.float16, device="cuda"), torch.full((M, N), 99, dtype=torch.int8, device="cuda")
    g.calls.gpusq_spgemm_int8_codes(dev(Xq), g.pack(dev(vals), dev(meta), K), dev(np.array([s_a])), dev(s_w), None if bias is None else dev(bias), Y, Yq,
                                    dev(np.array([s_y])), M, N, K, g.EPI_BIAS if biased else 0)
    assert np.array_equal(host(Y)[rows].view(np.uint16), y.view(np.uint16))
    assert np.array_equal(host(Yq)[rows], codes)


@pytest.mark.parametrize("kernel,M,N", [(4, 197, 192), (0, 300, 256), (2, 2048, 768)])
@pytest.mark.parametrize("at", [0, 64])
def test_codes_over_the_input(g, force_kernel, kernel, M, N, at):
    """Yq over Xq, whole or from a later row on: the same as with buffers of their own"""
    force_kernel(kernel)
    rng = np.random.default_rng(M)
    Xq = dev(rng.integers(-127, 128, (M, N)).astype(np.int8))
    _, s_w, vals, meta = _oracle_weights(synth.weights(N, N, seed=M, ids=(1,)))
    packed, scale = g.pack(dev(vals), dev(meta), N), dev(np.array([0.02, 0.05], np.float32))
    both = torch.zeros((M + at, N), dtype=torch.int8, device="cuda")
    both[:M] = Xq
    out = []
    for x, q in ((Xq, torch.empty_like(Xq)), (both[:M], both[at:])):
        Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
        g.calls.gpusq_spgemm_int8_codes(x, packed, scale[:1], dev(s_w), None, Y, q, scale[1:], M, N, N, 0)
        out.append((host(Y), host(q)))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("kernel,M,K,N", [(4, 33, 144, 132), (0, 65, 192, 68), (1, 129, 128, 256), (2, 1111, 512, 272), (2, 700, 272, 260)])
@pytest.mark.parametrize("scale", [0.0, -0.0, np.inf, -0.04, 1e-45, 1e-38, 3e38, np.nan])
def test_scales_and_outputs_that_leave_the_numbers(g, force_kernel, kernel, M, K, N, scale):
    """Zero, infinite, negative, denormal and no scales on outputs of which some are infinite and some are no numbers: the codes of the
    oracle's quantiser, and the output of gpusq_spgemm_int8"""
    force_kernel(kernel)
    Xq = dev(np.random.default_rng(M).integers(-127, 128, (M, K)).astype(np.int8))
    _, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=M, ids=(1,)))
    s_w[:8] = [np.nan, np.inf, -np.inf, 1e30, -1e30, 0.0, 1e-45, np.float32(6e-8)]
    bias = synth.bias(N, seed=M, ids=(2,))
    bias[8:12] = [np.nan, np.inf, -np.inf, 1e-40]
    packed, sa, sw, b = g.pack(dev(vals), dev(meta), K), dev(np.array([0.02], np.float32)), dev(s_w), dev(bias)
    y = g.spgemm_int8(Xq, packed, N, act_scale=sa, w_scale=sw, bias=b)
    assert torch.isnan(y).any() and torch.isinf(y).any()
    with np.errstate(all="ignore"):
        codes, _ = oracle.quantize_tensor_int8(host(y).astype(np.float32), scale=scale)
    Y, Yq = torch.full((M, N), 7.0, dtype=torch.float16, device="cuda"), torch.full((M, N), 99, dtype=torch.int8, device="cuda")
    g.calls.gpusq_spgemm_int8_codes(Xq, packed, sa, sw, b, Y, Yq, dev(np.array([scale], np.float32)), M, N, K, g.EPI_BIAS)
    assert np.array_equal(host(Y), host(y), equal_nan=True)
    assert np.array_equal(host(Yq), codes)


def test_infinite_outputs_and_refusals(g):
    """Outputs beyond fp16 and their codes; GELU is refused, and so is a missing scale."""
    M, K, N = 64, 128, 64
    Xq = np.full((M, K), 127, np.int8)
    _, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=1, ids=(1,)))
    acc = oracle.spgemm_int8(Xq, vals, meta)
    s_a = np.float32(1e6)
    with np.errstate(over="ignore"):
        y = oracle.epilogue_int8_f32(acc, float(s_a), s_w, None)["y16"]
    assert np.isinf(y).any()
    codes, _ = oracle.quantize_tensor_int8(y.astype(np.float32), scale=500.0)
    Y, Yq = torch.empty((M, N), dtype=torch.float16, device="cuda"), torch.empty((M, N), dtype=torch.int8, device="cuda")
    args = [dev(Xq), g.pack(dev(vals), dev(meta), K), dev(np.array([s_a])), dev(s_w), None, Y, Yq, dev(np.array([500.0], np.float32)), M, N, K, 0]
    g.calls.gpusq_spgemm_int8_codes(*args)
    assert np.array_equal(host(Y).view(np.uint16), y.view(np.uint16)) and np.array_equal(host(Yq), codes)
    for at, value in ((11, g.EPI_GELU), (7, None), (6, None)):
        with pytest.raises(g.GpusqError):
            g.calls.gpusq_spgemm_int8_codes(*(args[:at] + [value] + args[at + 1:]))
