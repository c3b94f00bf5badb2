"""The INT8 layer on the kernel that quantises whole rows of activations (wide.hip) against the CPU oracle: codes and scale of every row, the
first and last row of every slab of the output."""
import numpy as np
import pytest

import oracle
from paper_2305_10727_amd import synth
from test_gpu_parity import check_gelu_codes, dev, g, force_kernel, host, ulp_diff_f16, _oracle_weights  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (on 256 CUs) chunks of 1 row, of one slab less, whole and one row more, of every height, two and three rounds of chunks of two heights; one to twelve
# 64-channel blocks, the last partly outside, two and three column blocks, an uneven split with an idle wavefront; K of one piece, of one K
# step, of fewer steps than are in flight, odd and even numbers of them, ragged
SHAPES = [(1, 16, 16), (15, 128, 64), (16, 144, 80), (17, 384, 768), (4096, 512, 256), (5003, 272, 784), (8200, 640, 768), (12608, 768, 768), (16389, 400, 256), (20000, 128, 1040),
          (33000, 256, 528), (50000, 128, 128), (2500, 1296, 1552), (3000, 3088, 192)]


def _is_wide(g, dtype, out, M, K, N, gelu=False):
    return g.lib().gpusq_linear_int8_quantiser(g.F16 if dtype == np.float16 else g.F32, g._TORCH_DT[out], M, N, K, g.EPI_GELU if gelu else 0, 0, 0) == g.QUANTISE_WHOLE_ROWS


def _refined(s):
    """whether no reciprocal of the scale (rounded, the next above, below) decides all codes of fp16 values as the division does: for one of the
    two fp16 neighbours of a code boundary each of them fails"""
    s, c = np.float32(abs(s)), np.arange(254)
    if not 2.0 ** -100 <= s <= 2.0 ** 100:
        return False
    with np.errstate(over="ignore"):
        b = ((c >> 1).astype(np.float32) + np.float32(0.5)) * s
        down = b.astype(np.float16)
    bits = down.view(np.uint16).astype(np.int32) - (down.astype(np.float32) > b) + (c & 1)
    x = bits[bits < 0x7C00].astype(np.uint16).view(np.float16).astype(np.float32)
    exact, r = np.minimum(np.rint(x / s), 127), int((np.float32(1) / s).view(np.uint32))
    fma = lambda r: (x.astype(np.longdouble) * np.longdouble(np.uint32(r).view(np.float32)) + np.longdouble(12582912)).astype(np.float32)  # exact before it is rounded
    return all((np.minimum(fma(r + d) - np.float32(12582912), 127) != exact).any() for d in (0, 1, -1))


def _rows(M):
    m = np.arange(M)
    m = m[(m % 16 == 0) | (m % 16 == 15) | (m == M - 1)]
    return m if len(m) < 1500 else np.unique(np.concatenate([m[:400], m[-400:], m[::9]]))


def _layer(g, X, packed, sw, b, M, N, K, scale, out, out_scale, gelu):
    Y = torch.empty((M, N), dtype=out, device="cuda").fill_(7)
    Xq, sa, ws = torch.full((M, K), 99, dtype=torch.int8, device="cuda"), torch.zeros(1, device="cuda") if scale is None else scale, torch.empty(4096, dtype=torch.uint8, device="cuda")
    g.calls.gpusq_linear_int8(X, g._TORCH_DT[X.dtype], packed, sa, int(scale is not None), sw, b, Y, g._TORCH_DT[out], out_scale, Xq, ws, M, N, K, g._epi(b, gelu))
    return host(Y), host(Xq), host(sa)


@pytest.mark.parametrize("M,K,N", SHAPES)
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("given", [False, True])
def test_layer(g, force_kernel, M, K, N, dtype, given):
    force_kernel(5)
    assert all(_is_wide(g, dtype, out, M, K, N, gelu) for out in (torch.float16, torch.int8) for gelu in (False, True))
    assert g.lib().gpusq_linear_int8_launches(g.F16 if dtype == np.float16 else g.F32, M, N, K, g.EPI_BIAS, int(given), 0) == (1 if given else 2)
    rng = np.random.default_rng(M + K)
    X = (rng.standard_normal((M, K)) * 1.5).astype(dtype)
    if given:  # clamped, 0
        X.reshape(-1)[:8] = np.array([0.0, -0.0, 65504.0, -65504.0, 6e-8, np.inf, -np.inf, np.nan], dtype)
        X[-1, -2:] = np.array([np.nan, -np.inf], dtype)
    _, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=M, ids=(1,), sigma=0.05))
    bias, r = synth.bias(N, seed=M, ids=(2,)), _rows(M)
    packed, sw, b, x = g.pack(dev(vals), dev(meta), K), dev(s_w), dev(bias), dev(X)
    scale = np.float32(4.0 / 127.0) if given else None
    exp_q, exp_s = oracle.quantize_tensor_int8(X.astype(np.float32), scale=None if scale is None else float(scale))
    acc = oracle.spgemm_int8(exp_q[r], vals, meta)
    sa = lambda: None if scale is None else dev(np.array([scale]))
    y, q, s = _layer(g, x, packed, sw, b, M, N, K, sa(), torch.float16, None, False)
    assert s[0] == np.float32(exp_s) and np.array_equal(q, exp_q)
    assert np.array_equal(y[r].view(np.uint16), oracle.epilogue_int8_f32(acc, float(s[0]), s_w, bias)["y16"].view(np.uint16))
    y, q, _ = _layer(g, x, packed, sw, None, M, N, K, sa(), torch.float16, None, True)
    assert np.array_equal(q, exp_q) and ulp_diff_f16(y[r], oracle.epilogue_int8_f64(acc, float(s[0]), s_w, None, gelu=True)["y16"]).max() <= 1
    so = np.float32(np.abs(acc).max() * s[0] * s_w.max() / 100.0 + 1e-9)
    y, q, _ = _layer(g, x, packed, sw, b, M, N, K, sa(), torch.int8, dev(np.array([so])), False)
    assert np.array_equal(q, exp_q) and np.array_equal(y[r], oracle.epilogue_int8_f32(acc, float(s[0]), s_w, bias, out_scale=float(so))["q8"])
    y, _, _ = _layer(g, x, packed, sw, b, M, N, K, sa(), torch.int8, dev(np.array([so])), True)
    check_gelu_codes(y[r].astype(np.int32), acc, float(s[0]), s_w, bias, so)


# scales whose codes one fused multiply-add does not decide (eight of them), or whose quotients leave the numbers: every fp16 value
def test_codes(g, force_kernel):
    force_kernel(5)
    h = np.arange(0, 0x7C00, dtype=np.uint16).view(np.float16)
    X = np.concatenate([h, -h]).reshape(62, 1024)
    N, K = 16, 1024
    assert _is_wide(g, np.float16, torch.float16, 62, K, N)
    _, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=1))
    packed, sw, b = g.pack(dev(vals), dev(meta), K), dev(s_w), dev(synth.bias(N))
    rng = np.random.default_rng(3)
    scales = [np.float32(v) for v in (1.0, 1 / 3, 0.7, 3e-5, 5e-8, 511.5, 1e-38, 1e-45, 1e38, 0.0, np.inf, -0.25)]
    scales += [np.float32(np.float32(v) / np.float32(c + 0.5)) for v, c in zip(rng.uniform(0.5, 2.0, 40).astype(np.float16), rng.integers(0, 127, 40))]
    assert sum(_refined(s) for s in scales) >= 4
    for s in scales:
        with np.errstate(all="ignore"):
            exp, _ = oracle.quantize_tensor_int8(X.astype(np.float32), scale=float(s))
        assert np.array_equal(_layer(g, dev(X), packed, sw, b, 62, N, K, dev(np.array([s], np.float32)), torch.float16, None, False)[1], exp), s


# the scale of X's own range where X holds no, only tiny or not only numbers, or where no reciprocal decides: as from the quantiser and the GEMM
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("kind", ["nan", "inf", "both", "zero", "tiny", "all nan", "refined"])
def test_own_range(g, force_kernel, dtype, kind):
    M, K, N = 130, 272, 80
    X = (np.random.default_rng(5).standard_normal((M, K)) * {"zero": 0, "tiny": 1e-7}.get(kind, 1)).astype(dtype)
    for v, k in ((np.nan, ("nan", "both")), (np.inf, ("inf", "both")), (-np.inf, ("both",))):
        if kind in k: X.reshape(-1)[np.random.default_rng(len(k)).integers(0, M * K, 50)] = v
    if kind == "all nan": X[:] = np.nan
    if kind == "refined":  # a largest value whose scale is such a one, and values on its code boundaries
        amax = next(v for v in np.arange(0x4400, 0x4800, dtype=np.uint16).view(np.float16) if _refined(np.float32(v) / np.float32(127)))
        X = np.clip(X, -amax, amax).astype(dtype)
        X[0, :128] = (amax / np.float32(127) * (np.arange(128, dtype=np.float32) - np.float32(0.5))).astype(np.float16)
        X[0, 0] = amax
    _, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=M, ids=(9,), sigma=0.05))
    packed, sw, b, x = g.pack(dev(vals), dev(meta), K), dev(s_w), dev(synth.bias(N, seed=M, ids=(10,))), dev(X)
    q, s = g.quantize_int8(x, g.PER_TENSOR)
    exp = host(g.spgemm_int8(q, packed, N, act_scale=s, w_scale=sw, bias=b))
    force_kernel(5)
    assert _is_wide(g, dtype, torch.float16, M, K, N)
    y, codes, scale = _layer(g, x, packed, sw, b, M, N, K, None, torch.float16, None, False)
    assert np.array_equal(codes, host(q)) and np.array_equal(scale.view(np.uint32), host(s).view(np.uint32)) and np.array_equal(y, exp, equal_nan=True)


# Y over X, over the partial maxima of the range pass, out_scale the scale that the call finds: as from operands that lie apart
@pytest.mark.parametrize("how", ["input", "workspace", "scale"])
def test_shared_operands(g, force_kernel, how):
    M, K, N = 3000, 256, 256
    _, s_w, vals, meta = _oracle_weights(synth.weights(N, K, seed=M, ids=(7,), sigma=0.05))
    packed, sw, b = g.pack(dev(vals), dev(meta), K), dev(s_w), dev(synth.bias(N, seed=M, ids=(8,)))
    x = dev((np.random.default_rng(N).standard_normal((M, K)) * 1.5).astype(np.float16))
    q, s = g.quantize_int8(x, g.PER_TENSOR)
    out = torch.int8 if how == "scale" else torch.float16
    exp = g.spgemm_int8(q, packed, N, act_scale=s, w_scale=sw, bias=b, out_dtype=out, out_scale=s if how == "scale" else None)
    force_kernel(5)
    Xq, scale, ws = torch.empty((M, K), dtype=torch.int8, device="cuda"), torch.full((1,), 1e3, device="cuda"), torch.empty(4096, dtype=torch.uint8, device="cuda")
    Y = x.clone() if how == "input" else torch.empty((M, N), dtype=out, device="cuda")
    g.calls.gpusq_linear_int8(Y if how == "input" else x, g.F16, packed, scale, 0, sw, b, Y, g._TORCH_DT[out], scale if how == "scale" else None, Xq,
                              Y if how == "workspace" else ws, M, N, K, g.EPI_BIAS)
    assert torch.equal(Xq, q) and torch.equal(scale, s) and torch.equal(Y, exp)


# a size that the rules send there, recorded into a graph: replays between eager work on other inputs
def test_graph(g):
    from paper_2305_10727_amd.pipeline import SparseLinear
    M, K, N = 7029, 1152, 256
    assert g.lib().gpusq_linear_int8_launches(g.F16, M, N, K, g.EPI_BIAS, 0, 0) == 2
    lin = SparseLinear(M, K, N, "int8")
    lin.prepare_weights(dev(synth.weights(N, K, seed=5)))
    b, x = dev(synth.bias(N)), torch.empty((M, K), dtype=torch.float16, device="cuda")
    fill = lambda seed: x.copy_(dev(np.random.default_rng(seed).standard_normal((M, K)).astype(np.float16)))
    fill(0)
    lin.forward(x, b)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lin.forward(x, b)
    for seed in (1, 2, 3):
        fill(seed)
        y, q, s = lin.forward(x, b).clone(), lin.Xq.clone(), lin.act_scale.clone()
        exp_q, exp_s = g.quantize_int8(x, g.PER_TENSOR)
        assert torch.equal(q, exp_q) and torch.equal(s, exp_s)
        for t in (lin.Y, lin.Xq, lin.act_scale):
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(lin.Y, y) and torch.equal(lin.Xq, q) and torch.equal(lin.act_scale, s)


# layers that take the kernel by themselves below its many rows, or with more channels; rows of Y of no whole 16 channels, the last four in every place of a lane's
# eight and of a wavefront's 64, two column blocks, chunks that end inside a slab: as quantised and multiplied by two calls, bit for bit
@pytest.mark.parametrize("M,K,N", [(257, 64, 2560), (300, 256, 1936), (1000, 272, 528), (1024, 1024, 1040), (1301, 128, 1472), (2047, 512, 4096), (2048, 768, 1024),
                                   (1000, 128, 644), (1003, 192, 780), (9001, 320, 72), (9001, 576, 76), (5001, 384, 1500), (14070, 576, 252), (30000, 448, 212)])
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("out", [torch.float16, torch.int8])
def test_short_layer(g, M, K, N, dtype, out):
    assert _is_wide(g, dtype, out, M, K, N)
    r = torch.Generator(device="cuda").manual_seed(M)
    X = torch.randn((M, K), generator=r, device="cuda").to(torch.float16 if dtype == np.float16 else torch.float32)
    w = g.prepare_weights(torch.randn((N, K), generator=r, device="cuda") * 0.05, torch.int8)
    b, s = torch.randn(N, generator=r, device="cuda"), dev(np.array([0.03], np.float32))
    for given in (None, dev(np.array([0.025], np.float32))):
        Y, Xq, sa = _layer(g, X, w["packed"], w["w_scale"], b, M, N, K, given, out, s, False)
        q, sq = g.quantize_int8(X, g.PER_TENSOR, scale=given)
        assert np.array_equal(Xq, host(q)) and np.array_equal(sa, host(sq if given is None else given))
        ref = torch.empty((M, N), dtype=out, device="cuda")
        g.calls.gpusq_spgemm_int8(q, w["packed"], given if given is not None else sq, w["w_scale"], b, ref, g._TORCH_DT[out], s, M, N, K, g.EPI_BIAS)
        assert np.array_equal(Y.view(np.int16 if out == torch.float16 else np.int8), host(ref).view(np.int16 if out == torch.float16 else np.int8))
