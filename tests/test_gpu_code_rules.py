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


# scales under which values lie on code boundaries (0.03 ... 3/64), and others;
# negative scales decide as the division does too
@pytest.mark.parametrize("s", [0.03, 0.07, 0.7, 0.75, 3 / 64, 4 / 127, 1.0, 0.1, -0.03, -0.75, -3 / 64, -4 / 127])
def test_given_scale(g, force_kernel, s):
    for X in _every_fp16():
        exp, _ = oracle.quantize_tensor_int8(X.astype(np.float32), scale=float(np.float32(s)))
        for name, q in _codes_of_every_entry_point(g, force_kernel, X, s):
            assert np.array_equal(q, exp), name


def _reciprocals_that_agree(s):
    """Of the rounded 1 / s and the floats above and below it, which give every finite fp16 value the code of the division by one
    multiplication and one rounding to a whole number.  (The product of an fp16 value and a float is exact in 64 bits.)"""
    x = np.arange(0, 0x7C00, dtype=np.uint16).view(np.float16)
    exact = np.minimum(np.rint(x.astype(np.float32) / s), 127)
    r = np.float32(1) / s
    cand = (r, np.nextafter(r, np.float32(np.inf)), np.nextafter(r, np.float32(0)))
    return tuple(bool((np.minimum(np.rint(x.astype(np.float64) * np.float64(c)), 127) == exact).all()) for c in cand)


# a scale of each kind: the rounded reciprocal serves, only the one above or only the one below does, none (every product is refined)
@pytest.mark.parametrize("kind", ["rounded", "above", "below", "none"])
def test_reciprocal_next_to_the_rounded_one(g, force_kernel, kind):
    own = [np.float32(a) / np.float32(127) for a in np.arange(0x3C00, 0x4000, dtype=np.uint16).view(np.float16)]  # of amax in [1, 2)
    own += [np.float32(np.float32(v) / np.float32(c + 0.5)) for v, c in zip(np.linspace(0.5, 2, 200, dtype=np.float16), np.arange(200) % 127)]
    want = {"rounded": lambda a: a[0], "above": lambda a: not a[0] and a[1], "below": lambda a: not a[0] and not a[1] and a[2], "none": lambda a: not any(a)}[kind]
    scales = [s for s in own[::7] if want(_reciprocals_that_agree(s))][:4] or [s for s in own if want(_reciprocals_that_agree(s))][:4]
    assert scales
    for s in scales:
        for X in _every_fp16()[:2]:
            exp, _ = oracle.quantize_tensor_int8(X.astype(np.float32), scale=float(s))
            for name, q in _codes_of_every_entry_point(g, force_kernel, X, s):
                assert np.array_equal(q, exp), (name, s)
        # the scale of the data's own range
        top = np.float32(s) * np.float32(127)
        X = _every_fp16()[0].copy()
        X[np.abs(X.astype(np.float32)) > top] = 0
        exp_q, exp_s = oracle.quantize_tensor_int8(X.astype(np.float32))
        q, s_own = g.quantize_int8(dev(X), g.PER_TENSOR)
        assert host(s_own)[0] == np.float32(exp_s) and np.array_equal(host(q), exp_q)


# a scale by which quotients have no value (infinity by infinity, 0 by 0, NaN) or by which a finite value's product with the
# reciprocal overflows though its quotient is small
@pytest.mark.parametrize("s", [np.inf, -np.inf, np.nan, 0.0, -0.0, 1e-45, -1e-45, 3e-39, 1e38, 3.4e38])
def test_scale_without_a_reciprocal(g, force_kernel, s):
    for X in _every_fp16():
        with np.errstate(all="ignore"):
            exp, _ = oracle.quantize_tensor_int8(X.astype(np.float32), scale=float(np.float32(s)))
        for name, q in _codes_of_every_entry_point(g, force_kernel, X, s):
            assert np.array_equal(q, exp), name
    rng = np.random.default_rng(5)
    for cols in (1024, 1021):  # whole vectors; element by element
        X = (rng.integers(0, 2**32, (8, cols), dtype=np.uint64).astype(np.uint32)).view(np.float32).copy()  # every exponent
        X[1] *= np.float32(1e-38)  # denormals
        X[:, ::9], X[:, 4::9], X[::2, 7::9], X[:, 2::31] = np.inf, -np.inf, np.nan, 0.0
        with np.errstate(all="ignore"):
            exp, _ = oracle.quantize_tensor_int8(X, scale=float(np.float32(s)))
        given = np.float32(s)
        assert np.array_equal(host(g.quantize_int8(dev(X), g.PER_TENSOR, scale=dev(np.array([given])))[0]), exp)
        assert np.array_equal(host(g.quantize_int8(dev(X), g.PER_ROW, scale=dev(np.full(8, given)))[0]), exp)


# infinities in the data whose own range gives the scale: finite values 0, infinity by infinity 0
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("cols", [1024, 1021])
def test_range_with_infinities(g, dtype, cols):
    X = np.random.default_rng(6).standard_normal((9, cols)).astype(dtype)
    X[2, 5], X[4, 100], X[4, 900], X[7, ::3], X[8] = np.inf, -np.inf, np.nan, -np.inf, np.nan
    x, x32 = dev(X), X.astype(np.float32)
    with np.errstate(all="ignore"):
        for mode, ref in ((g.PER_ROW, oracle.quantize_rows_int8), (g.PER_TENSOR, lambda v: oracle.quantize_tensor_int8(v))):
            q, s = g.quantize_int8(x, mode)
            exp_q, exp_s = ref(x32)
            assert np.array_equal(host(q), exp_q) and np.array_equal(host(s), np.atleast_1d(np.asarray(exp_s, np.float32)))


def test_weights_with_infinities(g):
    W = (np.random.default_rng(7).standard_normal((70, 260)) * 0.02).astype(np.float32)
    W[3, 7], W[5, ::4], W[9, 250:] = np.inf, -np.inf, np.inf
    W[11] = W[11] * np.float32(1e-38)  # denormals: the scale's reciprocal is infinite
    out = g.prepare_weights(dev(W), torch.int8, want_intermediates=True)
    with np.errstate(all="ignore"):
        exp_q, exp_s = oracle.quantize_rows_int8(oracle.prune_2to4(W)[0])
    assert np.array_equal(host(out["w_scale"]), exp_s) and np.array_equal(host(out["W_low"]), exp_q)
    values, meta = oracle.compress(exp_q)[:2]
    assert np.array_equal(host(out["packed"]), host(g.pack(dev(values), dev(meta), 260)))


# given scales several times smaller than the row's own: quotients beyond 7 are clamped to it, so that the codes fit 4 bits
@pytest.mark.parametrize("cols", [1024, 1021, 5120])
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
def test_int4_rows_under_a_given_scale(g, dtype, cols):
    X = (np.random.default_rng(cols).standard_normal((9, cols)) * 3).astype(dtype)
    X[:, ::50], X[:, 7::50] = np.inf, -np.inf
    s = np.random.default_rng(8).uniform(0.02, 0.3, 9).astype(np.float32)
    exp, _ = oracle.quantize_rows_int4(X.astype(np.float32), scale=s)
    assert abs(exp).max() == 7
    assert np.array_equal(host(g.quantize_rows_int4(dev(X), scale=dev(s))[0]), exp)


# the per-tensor quantiser at the edges of its vectors (8 or 4 values), of its blocks (512 vectors) and of its grid (up to 1024
# workgroups, then several blocks to each, backwards in the second pass; fp16 beyond 96 MiB forwards)
@pytest.mark.parametrize("dtype,n", [(np.float16, n) for n in (1, 7, 8, 9, 4095, 4096, 4097, 4194304, 4194305, 4198401, 9000007, 50331656)]
                         + [(np.float32, n) for n in (1, 3, 4, 5, 2047, 2048, 2049, 2097152, 2097153, 2099201, 25165828)])
def test_per_tensor_quantiser_over_its_grid(g, dtype, n):
    X = (np.random.default_rng(n).standard_normal((1, n), dtype=np.float32) * 3).astype(dtype)
    X[0, n - 1] = dtype(40)  # the largest value last: in the scalar tail, or the last vector
    x = dev(X)
    exp_q, exp_s = oracle.quantize_tensor_int8(X.astype(np.float32))
    q, s = g.quantize_int8(x, g.PER_TENSOR)
    assert host(s)[0] == np.float32(exp_s) and np.array_equal(host(q), exp_q)
    given = np.float32(0.011)
    exp_q, _ = oracle.quantize_tensor_int8(X.astype(np.float32), scale=float(given))
    assert np.array_equal(host(g.quantize_int8(x, g.PER_TENSOR, scale=dev(np.array([given])))[0]), exp_q)


def _beside_boundaries(s):
    """Of one code and the next under the scale s, and values of other kinds"""
    h = (np.arange(-131, 131) + 0.5).astype(np.float32) * s
    steps = [h]
    for way in (np.float32(np.inf), np.float32(-np.inf)):
        v = h
        for _ in range(3):
            v = np.nextafter(v, way)
            steps.append(v)
    return np.concatenate(steps + [np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 3e38, -3e38, 1e-40, 6e4 * s, -6e4 * s], np.float32)])


# fp32 values on the boundaries between codes and up to 3 units in the last place beside them, through the fp32 quantiser and through
# every kernel's int8 output (zero activations: the value quantised is the bias); scales with a mantissa of ones, too small for
# the factor 65536 of the reciprocal, huge, negative, zero
@pytest.mark.parametrize("s", [0.03, 1 / 3, 4 / 127, 2.0 ** -7, float(np.nextafter(np.float32(0.5), np.float32(0))), -0.07, 1e-3, 3e-34, 1e-36, 1e30, 0.0])
def test_fp32_codes_beside_their_boundaries(g, force_kernel, s):
    s = np.float32(s)
    x = np.resize(_beside_boundaries(s), 2048).astype(np.float32)
    with np.errstate(all="ignore"):
        exp, _ = oracle.quantize_tensor_int8(x[None], scale=float(s))
    scale = dev(np.array([s]))
    assert np.array_equal(host(g.quantize_int8(dev(x[None]), g.PER_TENSOR, scale=scale)[0]), exp)
    K, one = 128, dev(np.ones(1, np.float32))
    for N in (2048, 2044):  # whole 16-byte pieces of int8; 4-byte ones
        packed = g.prepare_weights(torch.zeros((N, K), device="cuda"), torch.int8)["packed"]
        for M in (5, 300):
            X = torch.zeros((M, K), dtype=torch.int8, device="cuda")
            for kernel in (0, 1, 2, 3, 4):
                force_kernel(kernel)
                y = host(g.spgemm_int8(X, packed, N, act_scale=one, w_scale=torch.zeros(N, device="cuda"), bias=dev(x[:N]), out_dtype=torch.int8, out_scale=scale))
                assert np.array_equal(y, np.broadcast_to(exp[:, :N], (M, N))), (N, M, kernel)


# the same values as fp32 activations that the kernel for few rows quantises: their codes written out, and the operand itself (its
# product with the unit matrix); a workgroup of 4 wavefronts (2 K steps) and of 8 (5 steps, the last one short)
@pytest.mark.parametrize("s", [0.03, 1 / 3, 4 / 127, 2.0 ** -7, float(np.nextafter(np.float32(0.5), np.float32(0))), -0.07, 1e-3, 3e-34, 1e-36, 1e-45, 1e30, 0.0, -0.0,
                               np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("M,K", [(8, 256), (5, 560)])
def test_fp32_codes_beside_their_boundaries_inside_the_gemm(g, s, M, K):
    s = np.float32(s)
    X = np.resize(_beside_boundaries(s if np.isfinite(s) else np.float32(0.03)), M * K).astype(np.float32).reshape(M, K)
    with np.errstate(all="ignore"):
        exp, _ = oracle.quantize_tensor_int8(X, scale=float(s))
    assert g.lib().gpusq_linear_int8_launches(g.F32, M, K, K, 0, 1, 0) == 1
    packed = g.pack(*g.compress(torch.eye(K, dtype=torch.int8, device="cuda")), K)
    Y, Xq = torch.empty((M, K), dtype=torch.int32, device="cuda"), torch.full((M, K), 99, dtype=torch.int8, device="cuda")
    g.calls.gpusq_linear_int8(dev(X), g.F32, packed, dev(np.array([s])), 1, None, None, Y, g.I32, None, Xq, None, M, K, K, 0)
    assert np.array_equal(host(Xq), exp) and np.array_equal(host(Y), exp)
