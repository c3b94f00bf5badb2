"""Weight preparation at the sizes where its split over wavefronts changes: one wavefront per row up to 2048 elements (a batch of
512 groups in registers), four beyond, a second batch per lane beyond 8192; rows that end inside a K step, a packed lane or a
pair of groups, fewer rows than a fragment; kept weights that become zero codes.  Bit for bit against the separate calls, which
the parity tests hold against the oracle."""
import numpy as np
import pytest

from test_gpu_parity import dev, g, host  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [(5, 2044), (70, 2048), (300, 2052), (33, 4100), (9, 8188), (17, 8256), (4, 16384), (260, 1000)])
@pytest.mark.parametrize("dtype", ["int8", "fp16"])
def test_fused_preparation_equals_the_separate_calls(g, N, K, dtype):
    rng = np.random.default_rng(N + K)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    W[:, ::97] = 0.0
    W[0, : K // 2] = np.where(rng.random(K // 2) < 0.5, 1e-9, 0.0)  # kept values whose code (and fp16 rounding) is zero
    W[1 % N, 8:24] = np.repeat(np.float32([0.5, -0.5, 1e-6, 1e-6]), 4)
    tdt = torch.int8 if dtype == "int8" else torch.float16
    out = g.prepare_weights(dev(W), tdt, want_intermediates=True)
    Wp = g.prune_2to4(dev(W))
    Wl, s = g.quantize_int8(Wp, g.PER_ROW) if dtype == "int8" else (g.cast_f16(Wp), None)
    values, meta = g.compress(Wl)
    assert torch.equal(out["W_pruned"].view(torch.int32), Wp.view(torch.int32))
    assert torch.equal(out["W_low"], Wl) and torch.equal(out["values"], values) and torch.equal(out["meta"], meta)
    assert s is None or torch.equal(out["w_scale"], s)
    packed = g.pack(values, meta, K)
    assert torch.equal(out["packed"], packed)
    assert torch.equal(g.prepare_weights(dev(W), tdt)["packed"], packed)  # without the optional outputs


# only what the GEMM reads: 1 to 6 and 8 vectors of a row per lane, in one wavefront or four, several batches of 8; rows that end inside
# a lane, infinities and rows of zeros and denormals (whose scale has no reciprocal)
@pytest.mark.parametrize("N,K", [(1, 4), (12, 64), (70, 260), (33, 516), (300, 768), (40, 1028), (257, 1280), (8, 1540), (9, 1796), (30, 2052), (5, 3076), (70, 4096),
                                 (6, 5120), (3, 6148), (4, 7172), (5, 12292)])
@pytest.mark.parametrize("dtype", ["int8", "fp16"])
def test_packed_operand_and_scales_alone(g, N, K, dtype):
    rng = np.random.default_rng(N * 7 + K)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    W[0, ::3] = np.float32(1e-9)
    if N > 4:
        W[1], W[2] = 0.0, W[2] * np.float32(1e-38)
        W[3, 1], W[4, K // 2] = np.inf, -np.inf
    tdt = torch.int8 if dtype == "int8" else torch.float16
    out = g.prepare_weights(dev(W), tdt)
    Wp = g.prune_2to4(dev(W))
    Wl, s = g.quantize_int8(Wp, g.PER_ROW) if dtype == "int8" else (g.cast_f16(Wp), None)
    values, meta = g.compress(Wl)
    assert torch.equal(out["packed"], g.pack(values, meta, K))
    assert s is None or torch.equal(out["w_scale"], s)


@pytest.mark.parametrize("rows,cols", [(3, 2048), (5, 2052), (2, 5120), (7, 5124), (3, 1001), (1, 4)])
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_row_quantiser_batches(g, rows, cols, dtype):
    import oracle
    X = (np.random.default_rng(cols).standard_normal((rows, cols)) * 3).astype(dtype)
    q, s = g.quantize_int8(dev(X), g.PER_ROW)
    exp_q, exp_s = oracle.quantize_rows_int8(X.astype(np.float32))
    assert np.array_equal(host(q), exp_q) and np.array_equal(host(s), exp_s)


# rows of up to 1, 2, 4, 8 and 20 vectors per lane and more, of 4 and of 8 values, with their own and with given scales
@pytest.mark.parametrize("cols", [8, 64, 256, 264, 512, 516, 520, 768, 1024, 1032, 1280, 2048, 2056, 4096, 4104, 5120, 10240, 10248])
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_row_quantiser_vectors(g, cols, dtype):
    import oracle
    rng = np.random.default_rng(cols)
    X = (rng.standard_normal((6, cols)) * 3).astype(dtype)
    X[0, -1], X[1, 0] = 40, -40  # the ranges of two rows at their ends
    given = rng.uniform(0.02, 0.3, 6).astype(np.float32)
    for quantise, ref in ((lambda x, s: g.quantize_int8(x, g.PER_ROW, scale=s), oracle.quantize_rows_int8),
                          (lambda x, s: g.quantize_rows_int4(x, scale=s), oracle.quantize_rows_int4)):
        q, s = quantise(dev(X), None)
        exp_q, exp_s = ref(X.astype(np.float32))
        assert np.array_equal(host(q), exp_q) and np.array_equal(host(s), exp_s)
        assert np.array_equal(host(quantise(dev(X), dev(given))[0]), ref(X.astype(np.float32), scale=given)[0])
