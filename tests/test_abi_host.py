"""Host-only checks of the C-ABI library: it loads, exports every symbol the header declares, and rejects bad
arguments before touching the GPU.  No kernel is launched here."""
import ctypes
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "gpusq.h")
LIB = os.path.join(ROOT, "paper_2305_10727_amd", "libgpusq.so")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2305_10727_amd import build
        build.build()
    return ctypes.CDLL(LIB)


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(gpusq_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    names = declared_functions()
    assert len(names) >= 14
    for n in names:
        assert hasattr(lib, n), n
    from paper_2305_10727_amd import gpusq
    assert sorted(gpusq.EXPORTS) == names


def test_status_strings_and_version(lib):
    lib.gpusq_status_string.restype = ctypes.c_char_p
    seen = {lib.gpusq_status_string(i) for i in range(7)}
    assert len(seen) == 7 and lib.gpusq_status_string(0) == b"ok" and lib.gpusq_status_string(7) == b"unknown status"
    assert lib.gpusq_version() >= 100


def test_argument_errors_are_caught_on_the_host(lib):
    vp, i64, ci = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int
    OK, ERR_NULL, ERR_SHAPE, ERR_ALIGN, ERR_UNSUPPORTED = 0, 1, 2, 3, 4
    good = vp(0x10000)  # never dereferenced: every call below fails validation first
    odd = vp(0x10008)
    lib.gpusq_prune_2to4.argtypes = [vp, vp, vp, ci, i64, i64, vp]
    assert lib.gpusq_prune_2to4(None, good, None, 0, 4, 8, None) == ERR_NULL
    assert lib.gpusq_prune_2to4(good, good, None, 0, 4, 6, None) == ERR_SHAPE
    assert lib.gpusq_prune_2to4(good, good, None, 0, 0, 8, None) == ERR_SHAPE
    assert lib.gpusq_prune_2to4(good, good, None, 2, 4, 8, None) == ERR_UNSUPPORTED
    assert lib.gpusq_prune_2to4(odd, good, None, 0, 4, 8, None) == ERR_ALIGN
    lib.gpusq_compress.argtypes = [vp, vp, vp, vp, ci, i64, i64, vp]
    assert lib.gpusq_compress(good, good, None, None, 1, 4, 8, None) == ERR_NULL
    assert lib.gpusq_compress(good, good, good, None, 0, 4, 8, None) == ERR_UNSUPPORTED
    assert lib.gpusq_compress(good, good, good, None, 1, 4, 10, None) == ERR_SHAPE
    lib.gpusq_check_2to4.argtypes = [vp, ci, vp, i64, i64, vp]
    assert lib.gpusq_check_2to4(good, 0, None, 4, 8, None) == ERR_NULL          # the counter is required
    assert lib.gpusq_check_2to4(good, 3, good, 4, 8, None) == ERR_UNSUPPORTED   # int32 tensors
    assert lib.gpusq_check_2to4(good, 0, good, 4, 6, None) == ERR_SHAPE
    assert lib.gpusq_check_2to4(odd, 0, good, 4, 8, None) == ERR_ALIGN
    assert lib.gpusq_check_2to4(good, 0, vp(0x10002), 4, 8, None) == ERR_ALIGN
    lib.gpusq_quantize_int8.argtypes = [vp, ci, vp, vp, ci, ci, i64, i64, vp, vp]
    assert lib.gpusq_quantize_int8(good, 0, good, None, 0, 0, 4, 8, None, None) == ERR_NULL
    assert lib.gpusq_quantize_int8(good, 0, good, good, 1, 0, 4, 8, None, None) == ERR_NULL  # per-tensor needs workspace
    assert lib.gpusq_quantize_int8(good, 0, good, good, 7, 0, 4, 8, good, None) == ERR_UNSUPPORTED
    assert lib.gpusq_quantize_int8(good, 0, good, good, 0, 0, -1, 8, good, None) == ERR_SHAPE
    lib.gpusq_spgemm_int8.argtypes = [vp, vp, vp, vp, vp, vp, ci, vp, i64, i64, i64, ci, vp]
    assert lib.gpusq_spgemm_int8(good, good, None, None, None, good, 3, None, 8, 8, 24, 0, None) == ERR_UNSUPPORTED  # K % 16
    assert lib.gpusq_spgemm_int8(good, good, None, None, None, good, 3, None, 8, 6, 32, 0, None) == ERR_UNSUPPORTED  # N % 4
    assert lib.gpusq_spgemm_int8(good, good, None, None, None, good, 3, None, 8, 8, 30, 0, None) == ERR_SHAPE
    assert lib.gpusq_spgemm_int8(good, good, None, None, None, good, 1, None, 8, 8, 32, 0, None) == ERR_NULL  # scales
    assert lib.gpusq_spgemm_int8(good, good, good, good, None, good, 1, None, 8, 8, 32, 1, None) == ERR_NULL  # bias flag
    assert lib.gpusq_spgemm_int8(good, good, good, good, None, good, 2, None, 8, 8, 32, 0, None) == ERR_NULL  # out_scale
    assert lib.gpusq_spgemm_int8(good, good, good, good, None, good, 1, None, 8, 8, 32, 8, None) == ERR_UNSUPPORTED
    # fp16 activations quantised inside the GEMM: the same checks, and problems of the tile kernel are refused
    lib.gpusq_spgemm_int8_xf16.argtypes = [vp, vp, vp, vp, vp, vp, ci, vp, i64, i64, i64, ci, vp]
    assert lib.gpusq_spgemm_int8_xf16(good, good, None, None, None, good, 1, None, 8, 8, 32, 0, None) == ERR_NULL  # scales
    assert lib.gpusq_spgemm_int8_xf16(good, good, good, good, None, good, 2, None, 8, 8, 32, 0, None) == ERR_NULL  # out_scale
    # the scale quantises X, so it is required for raw accumulators as well
    assert lib.gpusq_spgemm_int8_xf16(good, good, None, None, None, good, 3, None, 8, 8, 32, 0, None) == ERR_NULL
    assert lib.gpusq_spgemm_int8_xf16(good, good, good, good, None, odd, 1, None, 8, 8, 32, 0, None) == ERR_ALIGN
    assert lib.gpusq_spgemm_int8_xf16(good, good, good, good, None, good, 1, None, 12608, 3072, 768, 0, None) == ERR_UNSUPPORTED
    lib.gpusq_spgemm_fp16.argtypes = [vp, vp, vp, vp, i64, i64, i64, ci, vp]
    assert lib.gpusq_spgemm_fp16(good, None, None, good, 8, 8, 32, 0, None) == ERR_NULL
    assert lib.gpusq_spgemm_fp16(good, good, None, odd, 8, 8, 32, 0, None) == ERR_ALIGN
    assert lib.gpusq_spgemm_fp16(good, good, None, good, 0, 8, 32, 0, None) == ERR_SHAPE
    lib.gpusq_im2col_patches.argtypes = [vp, vp, ci, i64, i64, i64, i64, i64, i64, vp]
    assert lib.gpusq_im2col_patches(good, None, 2, 1, 3, 32, 32, 16, 768, None) == ERR_NULL
    assert lib.gpusq_im2col_patches(good, good, 2, 1, 3, 30, 32, 16, 768, None) == ERR_SHAPE   # H % P
    assert lib.gpusq_im2col_patches(good, good, 2, 1, 3, 32, 32, 16, 700, None) == ERR_SHAPE   # K_pad < C*P*P
    assert lib.gpusq_im2col_patches(good, good, 0, 1, 3, 32, 32, 16, 768, None) == ERR_UNSUPPORTED
    assert lib.gpusq_im2col_patches(odd, good, 2, 1, 3, 32, 32, 16, 768, None) == ERR_ALIGN
    lib.gpusq_patch_embed16_int8.argtypes = [vp, vp, vp, vp, vp, vp, i64, i64, i64, i64, i64, ci, vp]
    assert lib.gpusq_patch_embed16_int8(good, good, None, good, None, good, 4, 3, 224, 224, 768, 0, None) == ERR_NULL
    assert lib.gpusq_patch_embed16_int8(good, good, good, good, None, good, 4, 3, 220, 224, 768, 0, None) == ERR_SHAPE
    assert lib.gpusq_patch_embed16_int8(good, good, good, good, None, good, 4, 3, 224, 224, 768, 2, None) == ERR_UNSUPPORTED  # GELU
    assert lib.gpusq_patch_embed16_int8(good, good, good, good, None, good, 1, 3, 32, 32, 64, 0, None) == ERR_UNSUPPORTED   # too small
    lib.gpusq_patch_embed16_fp16.argtypes = [vp, vp, vp, vp, i64, i64, i64, i64, i64, ci, vp]
    assert lib.gpusq_patch_embed16_fp16(good, good, None, good, 4, 3, 224, 224, 768, 1, None) == ERR_NULL                  # bias flag
    lib.gpusq_prune_n_of_m.argtypes = [vp, vp, ci, ci, i64, i64, vp]
    assert lib.gpusq_prune_n_of_m(good, None, 1, 4, 4, 16, None) == ERR_NULL
    assert lib.gpusq_prune_n_of_m(good, good, 1, 5, 4, 20, None) == ERR_UNSUPPORTED   # m
    assert lib.gpusq_prune_n_of_m(good, good, 4, 4, 4, 16, None) == ERR_SHAPE         # n < m
    assert lib.gpusq_prune_n_of_m(good, good, 2, 16, 4, 24, None) == ERR_SHAPE        # K % m
    lib.gpusq_prune_4to8_pairs.argtypes = [vp, vp, vp, ci, i64, i64, vp]
    assert lib.gpusq_prune_4to8_pairs(good, None, None, 0, 4, 8, None) == ERR_NULL
    assert lib.gpusq_prune_4to8_pairs(good, good, None, 1, 4, 12, None) == ERR_SHAPE   # K % 8
    assert lib.gpusq_prune_4to8_pairs(odd, good, None, 0, 4, 8, None) == ERR_ALIGN
    lib.gpusq_int4_to_sparse_int8.argtypes = [vp, vp, vp, vp, vp, i64, i64, vp]
    assert lib.gpusq_int4_to_sparse_int8(good, good, good, None, None, 4, 8, None) == ERR_NULL
    assert lib.gpusq_int4_to_sparse_int8(good, good, good, good, None, 4, 12, None) == ERR_SHAPE
    assert lib.gpusq_int4_to_sparse_int8(good, good, odd, good, None, 4, 8, None) == ERR_ALIGN
    lib.gpusq_quantize_rows_int4.argtypes = [vp, ci, vp, vp, ci, i64, i64, vp]
    assert lib.gpusq_quantize_rows_int4(good, 0, good, None, 0, 4, 8, None) == ERR_NULL
    assert lib.gpusq_quantize_rows_int4(good, 2, good, good, 0, 4, 8, None) == ERR_UNSUPPORTED
    assert lib.gpusq_quantize_rows_int4(good, 0, good, good, 0, 0, 8, None) == ERR_SHAPE
    lib.gpusq_compress_int4.argtypes = [vp, vp, vp, vp, i64, i64, vp]
    assert lib.gpusq_compress_int4(good, good, None, None, 4, 8, None) == ERR_NULL
    assert lib.gpusq_compress_int4(good, good, good, None, 4, 20, None) == ERR_SHAPE
    lib.gpusq_decompress_int4.argtypes = [vp, vp, vp, i64, i64, vp]
    assert lib.gpusq_decompress_int4(good, good, None, 4, 8, None) == ERR_NULL
    assert lib.gpusq_decompress_int4(good, odd, good, 4, 8, None) == ERR_ALIGN
    lib.gpusq_packed_bytes.restype = ctypes.c_size_t
    lib.gpusq_packed_bytes.argtypes = [ci, i64, i64]
    # tiles of 256 channels x one 128-byte K step: 16 fragments of 1024 value bytes + 16 x 64 lanes of index bytes
    assert lib.gpusq_packed_bytes(2, 768, 192) == 3 * 2 * (16384 + 4096)
    assert lib.gpusq_packed_bytes(1, 768, 192) == 3 * 3 * (16384 + 2048)
    assert lib.gpusq_packed_bytes(2, 100, 144) == 1 * 2 * (16384 + 4096)
    assert lib.gpusq_packed_bytes(0, 768, 192) == 0 and lib.gpusq_packed_bytes(2, 768, 190) == 0
    lib.gpusq_quantize_workspace_bytes.restype = ctypes.c_size_t
    lib.gpusq_quantize_workspace_bytes.argtypes = [ci, i64, i64]
    assert lib.gpusq_quantize_workspace_bytes(0, 10, 10) == 0 and lib.gpusq_quantize_workspace_bytes(1, 10, 10) >= 4


def test_binding_refuses_host_tensors():
    torch = pytest.importorskip("torch")
    from paper_2305_10727_amd import gpusq
    with pytest.raises(ValueError):
        gpusq.prune_2to4(torch.zeros(4, 8))


def test_binding_refuses_addresses():
    """The checked calls take tensors: an integer is none and must not reach the GPU as an address."""
    pytest.importorskip("torch")
    from paper_2305_10727_amd import gpusq
    with pytest.raises(AttributeError):
        gpusq.calls.gpusq_cast_f16(4096, None, 16)
    with pytest.raises(AttributeError):
        gpusq.calls.gpusq_cast_f16(None, True, 16)


def _plan(lib, dt, M, N, K, epi, cus):
    out = (ctypes.c_int32 * 8)()
    lib.gpusq_spgemm_plan.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int,
                                      ctypes.POINTER(ctypes.c_int32)]
    st = lib.gpusq_spgemm_plan(dt, M, N, K, epi, cus, out)
    return st, list(out)


@pytest.mark.parametrize("dt,M,N,K", [(2, 1847, 972, 17920000), (2, 2807, 608, 17920000), (1, 3063, 884, 16777216), (1, 810, 3744, 8960000)])
def test_long_rows_beyond_the_tile_kernels_offsets_stay_with_the_small_kernel(lib, dt, M, N, K):
    """255 rows of K bytes past 2^32: kernel 2 refuses them, so what the 64 x 64 tiles took has to go on going there."""
    assert 255 * K * (1 if dt == 2 else 2) + 128 >= 2 ** 32
    st, p = _plan(lib, dt, M, N, K, 0, 256)
    assert st == 0 and p[0] == 0


def test_tile_plan_covers_every_row_exactly_once(lib):
    """The host-side tile plan of the sparse GEMM: the full tiles and the tail tiles partition the rows of X, the tile
    count is consistent, no more workgroups than tiles or compute units (rounded to the 8 XCDs), and a small problem
    takes the small kernel."""
    I8, F16 = 2, 1
    shapes = [(12608, 3072, 768), (25216, 768, 3072), (12544, 512, 2048), (65792, 5120, 1280), (50432, 1024, 4096),
              (600, 512, 384), (1500, 388, 256), (2100, 520, 128), (12345, 264, 128), (70000, 256, 128), (257, 1024, 1024),
              (3, 100000, 256), (999999, 4, 128)]
    for cus in (256, 64, 304, 8):
        for dt in (I8, F16):
            for epi in (0, 3):
                for M, N, K in shapes:
                    st, p = _plan(lib, dt, M, N, K, epi, cus)
                    assert st == 0, (M, N, K)
                    kernel, u, tiles_n, ftm, fchunks, ttm, total, wgs = p
                    if M * N <= 256 * 1024:
                        assert kernel == 0
                        continue
                    assert kernel in (0, 2, 3)
                    if kernel == 0:  # few rows: the estimated run times favour the small kernel
                        assert p[1:] == [0] * 7 and -(-M // 64) * -(-N // 64) <= 16 * cus
                        continue
                    # kernel 2: one workgroup per CU, tiles of up to 256 rows; kernel 3: two per CU, up to 128 rows
                    unit, max_tm, per_cu = (32, 8, 1) if kernel == 2 else (64, 2, 2)
                    assert u == unit and tiles_n == -(-N // 256)
                    assert 1 <= ftm <= max_tm and 1 <= ttm <= max_tm and fchunks >= 0
                    full_rows = fchunks * u * ftm
                    assert full_rows - u * ftm < M          # no full tile lies entirely beyond M
                    rows_left = max(M - full_rows, 0)
                    tail_chunks = -(-rows_left // (u * ttm))
                    assert total == (fchunks + tail_chunks) * tiles_n
                    assert full_rows + tail_chunks * u * ttm >= M                # every row is covered
                    assert tail_chunks == 0 or full_rows + (tail_chunks - 1) * u * ttm < M  # and no tail tile is empty
                    assert wgs % 8 == 0 and wgs <= -(-per_cu * cus // 8) * 8 and wgs >= min(total, 8) and wgs - 8 < total
    # one image (M = 197) takes the small kernel, a batch of 64 the tile kernel
    for N, K in ((2304, 768), (3072, 768), (768, 3072), (768, 768)):
        assert _plan(lib, I8, 197, N, K, 0, 256)[1][0] == 0 and _plan(lib, I8, 12608, N, K, 0, 256)[1][0] in (2, 3)
        assert _plan(lib, F16, 197, N, K, 0, 256)[1][0] == 0 and _plan(lib, F16, 12608, N, K, 0, 256)[1][0] in (2, 3)
    # beyond the few rows whose kernel splits K over its wavefronts the estimates decide again (fp16: 6 tiles of 32 rows to a CU)
    assert _plan(lib, F16, 1344, 2304, 3072, 1, 256)[1][0] == 2 and _plan(lib, F16, 4096, 768, 1536, 1, 256)[1][0] == 2
    # between the two tile kernels: wide, GELU and long-K layers stay on the one-workgroup kernel, layers with few output
    # channels, short K and no GELU take the kernel with two workgroups per CU
    assert _plan(lib, I8, 12608, 3072, 768, 3, 256)[1][0] == 2 and _plan(lib, I8, 25216, 768, 3072, 1, 256)[1][0] == 2
    assert _plan(lib, F16, 12608, 3072, 768, 3, 256)[1][0] == 2 and _plan(lib, F16, 50432, 1024, 4096, 1, 256)[1][0] == 2
    assert _plan(lib, I8, 25216, 768, 768, 1, 256)[1][0] == 3 and _plan(lib, F16, 12544, 1536, 512, 1, 256)[1][0] == 3
    assert _plan(lib, F16, 25216, 768, 768, 1, 256)[1][0] == 2  # FP16: only from 1024 output channels on
    # ragged K (not a multiple of the 128-byte K step): the tile kernel with one workgroup per CU takes it, the other does not;
    # argument errors are reported
    assert _plan(lib, I8, 4096, 4096, 144, 0, 256) == _plan(lib, I8, 4096, 4096, 256, 0, 256) == (0, [2, 32, 16, 8, 16, 8, 256, 256])
    assert _plan(lib, F16, 4096, 4096, 64, 0, 256)[1][0] == 2 and _plan(lib, F16, 4096, 4096, 80, 0, 256)[1][0] == 2
    assert _plan(lib, I8, 25216, 768, 784, 1, 256)[1][0] == 2
    assert _plan(lib, I8, 0, 4096, 128, 0, 256)[0] == 2 and _plan(lib, I8, 128, 4096, 130, 0, 256)[0] == 2
    assert _plan(lib, 0, 128, 4096, 128, 0, 256)[0] == 4 and _plan(lib, I8, 128, 4098, 128, 0, 256)[0] == 4


def test_force_kernel_override_is_an_explicit_call(lib):
    """the testing override: set and cleared through the ABI (no environment lookup per launch), visible in the plan query"""
    lib.gpusq_force_kernel.argtypes = [ctypes.c_int]
    I8 = 2
    prev = lib.gpusq_force_kernel(-1)
    try:
        assert _plan(lib, I8, 12608, 3072, 768, 0, 256)[1][0] == 2
        assert lib.gpusq_force_kernel(0) == -1
        assert _plan(lib, I8, 12608, 3072, 768, 0, 256)[1][0] == 0
        assert lib.gpusq_force_kernel(2) == 0
        assert _plan(lib, I8, 197, 768, 768, 0, 256)[1][0] == 2
        assert _plan(lib, I8, 197, 768, 144, 0, 256)[1][0] == 2
        assert lib.gpusq_force_kernel(3) == 2
        assert _plan(lib, I8, 197, 768, 144, 0, 256)[1][0] == 0   # ragged K cannot run on kernel 3: the rules decide
        assert _plan(lib, I8, 12608, 3072, 768, 0, 256)[1][0] == 3
        # 5: the size rules, but the layer on the kernel for whole rows at every size it can, those of the kernel for few rows among them
        assert lib.gpusq_force_kernel(5) == 3
        for M, N, K in ((1, 16, 16), (130, 80, 272), (62, 16, 1024), (17, 768, 384), (2048, 64, 256), (12608, 3072, 768)):
            for x_dt in (0, 1):
                assert lib.gpusq_linear_int8_quantiser(x_dt, 1, ctypes.c_int64(M), ctypes.c_int64(N), ctypes.c_int64(K), 0, 0, 256) == 2
                assert lib.gpusq_linear_int8_launches(x_dt, ctypes.c_int64(M), ctypes.c_int64(N), ctypes.c_int64(K), 0, 0, 256) == 2
        assert lib.gpusq_linear_int8_quantiser(1, 1, ctypes.c_int64(130), ctypes.c_int64(84), ctypes.c_int64(272), 0, 0, 256) == 1  # N % 16
        assert _plan(lib, I8, 12608, 3072, 768, 0, 256)[1][0] == 2
        assert lib.gpusq_force_kernel(3) == 5
        assert lib.gpusq_force_kernel(7) == 3                      # anything else clears the override
        assert lib.gpusq_force_kernel(-1) == -1
    finally:
        lib.gpusq_force_kernel(prev)


def test_gelu_fit_stays_within_its_stated_bound_of_the_exact_function():
    """The epilogue's GELU (a polynomial fit in fp32, csrc/epilogue.h) against the oracle's erf form in fp64, over every
    finite fp16 argument and a dense fp32 grid: the difference stays below the stated 0.15 units in the last place of the
    exact value as an fp16 number.  The GPU tests build their element-wise code check on this bound."""
    np = pytest.importorskip("numpy")
    import oracle
    import gelu_fit
    h = np.arange(0, 0x7C00, dtype=np.uint16).view(np.float16).astype(np.float32)
    x = np.concatenate([np.linspace(-14.0, 14.0, 2000001).astype(np.float32), h, -h])
    exact = oracle.epilogue_fp16_f64(x.astype(np.float64).reshape(1, -1), None, True)["ref"][0]
    err = np.abs(gelu_fit.gelu_fit_f32(x).astype(np.float64) - exact) / gelu_fit.ulp16(exact)
    assert 0.05 < err.max() <= gelu_fit.FIT_BOUND_ULP16
    # so a rounded fp16 output is within one unit of the exact value's rounding, and a re-quantised code moves only at a tie
    assert np.isfinite(gelu_fit.gelu_fit_f32(np.array([-65504.0, 65504.0, 0.0, -0.0], np.float32))).all()


def test_every_tile_of_the_one_workgroup_kernel_is_met_once(tmp_path):
    """The plans of tile kernel 2 walked on the host with the code the kernel reads them with (tile_plan_walk.cpp), over random sizes
    and several numbers of compute units"""
    exe = str(tmp_path / "walk")
    build = subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                            "-I", os.path.join(ROOT, "paper_2305_10727_amd", "csrc"), os.path.join(ROOT, "tests", "tile_plan_walk.cpp"), "-o", exe],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([exe, "20000"], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout == "20000 plans\n", run.stdout


def test_launch_rules(tmp_path):
    """The grid of the pair-wise pruning kernel and the question whether a GEMM may quantise its own activations, by the code the
    library launches with (launch_rules_walk.cpp)"""
    exe = str(tmp_path / "rules")
    build = subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2305_10727_amd", "csrc"),
                            os.path.join(ROOT, "tests", "launch_rules_walk.cpp"), "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout == "ok\n", run.stdout


def test_every_chunk_of_the_kernel_for_whole_rows_is_met_once(tmp_path):
    """The plans of the kernel that quantises whole rows walked on the host with the code the kernel reads them with (wide_plan_walk.cpp)"""
    exe = str(tmp_path / "walk")
    build = subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                            "-I", os.path.join(ROOT, "paper_2305_10727_amd", "csrc"), os.path.join(ROOT, "tests", "wide_plan_walk.cpp"), "-o", exe],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([exe, "20000"], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout == "20000 plans\n", run.stdout


def test_walk_block_mlp_plans(tmp_path):
    """The plans of the kernel for the layers behind attention, walked on the host with the code the kernel reads them with (mlp_plan_walk.cpp)"""
    exe = str(tmp_path / "walk")
    build = subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                            "-I", os.path.join(ROOT, "paper_2305_10727_amd", "csrc"), os.path.join(ROOT, "tests", "mlp_plan_walk.cpp"), "-o", exe],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([exe, "20000"], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout == "20000 plans\n", run.stdout


def test_walk_patch_embedding_plans(tmp_path):
    """The plans of the kernel for patch embeddings, and where it keeps their values, walked on the host with the code the kernel uses (patches_plan_walk.cpp)"""
    exe = str(tmp_path / "walk")
    build = subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                            "-I", os.path.join(ROOT, "paper_2305_10727_amd", "csrc"), os.path.join(ROOT, "tests", "patches_plan_walk.cpp"), "-o", exe],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([exe, "20000"], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout == "20000 plans\n", run.stdout


@pytest.mark.parametrize("sizes,launches", [
    ((256, 3, 224, 224, 14, 640, 1280, 1), 1), ((3, 3, 224, 224, 14, 592, 512, 0), 1), ((64, 3, 224, 224, 14, 640, 2048, 1), 1),
    ((2, 3, 224, 224, 14, 640, 128, 1), 2),     # fewer than 640 patches
    ((12, 3, 224, 224, 14, 640, 1088, 1), 2),   # too few for the weights: 3072 patches, 1088 channels
    ((64, 3, 252, 252, 18, 976, 512, 1), 1), ((64, 3, 252, 252, 18, 976, 576, 1), 2),  # LDS for two slabs: up to 512 channels,
    ((10, 3, 252, 252, 18, 976, 512, 1), 2),                                           # from 2048 patches on
    ((64, 3, 224, 224, 28, 2368, 192, 1), 2),   # LDS for one slab
    ((64, 3, 224, 224, 16, 768, 768, 1), 2), ((4, 3, 224, 224, 16, 768, 192, 1), 2),  # 16-byte pieces
    ((64, 3, 225, 225, 15, 704, 768, 1), 2),    # no pairs of pixels
    ((64, 3, 224, 224, 14, 640, 776, 1), 2),    # part of a block of channels
    ((64, 3, 224, 224, 14, 640, 768, 3), 2),    # GELU
    ((2, 3, 32760, 32760, 14, 640, 768, 1), 2), # images of 4 GiB or more
    ((1, 3, 225, 224, 14, 640, 768, 1), 0), ((1, 3, 224, 224, 14, 580, 768, 1), 0), ((1, 3, 224, 224, 14, 640, 770, 1), 0), ((0, 3, 224, 224, 14, 640, 768, 1), 0)])
def test_patch_embedding_launches(sizes, launches):
    from paper_2305_10727_amd import gpusq
    assert gpusq.lib().gpusq_patch_embed_fp16_launches(*sizes, 256) == launches


# sizes that were timed slower in one launch, and neighbours that were timed faster
@pytest.mark.parametrize("sizes,launches", [
    ((11, 320, 44, 20, 2, 1280, 64, 1), 2), ((9, 32, 128, 128, 4, 512, 192, 1), 2), ((10, 8, 300, 300, 10, 832, 512, 1), 2),  # many channels
    ((9, 3, 128, 128, 4, 64, 192, 1), 1), ((10, 4, 300, 300, 10, 448, 512, 1), 1),
    ((39, 1, 192, 296, 8, 64, 2752, 1), 2), ((64, 3, 224, 224, 14, 640, 2176, 1), 2),                       # many channels out
    ((19, 2, 288, 306, 18, 704, 1152, 1), 2), ((1, 2, 640, 640, 20, 832, 576, 1), 2), ((32, 2, 288, 324, 18, 704, 1152, 1), 1),  # LDS for three slabs, with fewer and with them
    ((1, 1, 672, 672, 24, 576, 576, 1), 2), ((4, 1, 672, 672, 24, 576, 576, 1), 1),                         # few patches
    ((19, 3, 396, 720, 18, 1024, 384, 1), 2), ((15, 3, 396, 720, 18, 1024, 384, 1), 1), ((24, 3, 396, 720, 18, 1024, 384, 1), 1)])  # two slabs: workgroups just past a round, fewer, more
def test_patch_embeddings_timed_slower_in_one_launch_are_two(sizes, launches):
    from paper_2305_10727_amd import gpusq
    assert gpusq.lib().gpusq_patch_embed_fp16_launches(*sizes, 256) == launches


# four channels of the images and more than 256 out: from 800 patches on
@pytest.mark.parametrize("sizes,launches", [((3, 4, 160, 88, 8, 256, 384, 1), 2), ((25, 4, 210, 28, 14, 832, 320, 1), 2), ((3, 4, 160, 88, 8, 256, 256, 1), 1), ((3, 3, 160, 88, 8, 192, 384, 1), 1),
                                            ((4, 4, 160, 88, 8, 256, 384, 1), 1)])
def test_patch_embeddings_of_four_channels_timed_slower_in_one_launch_are_two(sizes, launches):
    from paper_2305_10727_amd import gpusq
    assert gpusq.lib().gpusq_patch_embed_fp16_launches(*sizes, 256) == launches


@pytest.mark.parametrize("sizes,launches", [
    ((256, 3, 224, 224, 14, 640, 1280, 1), 2), ((1, 3, 14, 14, 14, 592, 512, 0), 2), ((2, 3, 56, 56, 8, 192, 256, 1), 2),
    ((4, 3, 224, 224, 14, 640, 1088, 1), 4),    # too few for the weights: 1024 patches, 1088 channels
    ((16, 3, 224, 224, 14, 640, 1536, 1), 4),   # beyond 1408 channels 6 patches for each from 512 on, not 2
    ((64, 3, 224, 224, 16, 768, 768, 1), 4), ((1, 3, 224, 224, 16, 768, 772, 1), 2), ((1, 3, 224, 224, 16, 768, 768, 3), 4),  # 16 x 16: few of them, on the kernel for whole rows
    ((1, 3, 224, 224, 16, 784, 768, 1), 4), ((1, 4, 224, 224, 16, 1024, 768, 1), 2), ((1, 5, 224, 224, 16, 1280, 768, 1), 4), ((64, 3, 252, 252, 18, 1024, 256, 1), 4),  # more than 14 rows
    ((64, 9, 224, 224, 14, 1792, 192, 1), 4),   # LDS for fewer than three slabs
    ((64, 3, 225, 225, 15, 704, 768, 1), 4), ((64, 3, 224, 224, 14, 640, 776, 1), 4), ((64, 3, 224, 224, 14, 640, 768, 3), 4),
    ((2, 3, 32760, 32760, 14, 640, 768, 1), 0), # more pixels than the quantiser has columns
    ((1, 3, 225, 224, 14, 640, 768, 1), 0), ((1, 3, 224, 224, 14, 640, 770, 1), 0)])
def test_int8_patch_embedding_launches(sizes, launches):
    from paper_2305_10727_amd import gpusq
    for dt in (gpusq.F16, gpusq.F32):
        assert gpusq.lib().gpusq_patch_embed_int8_launches(dt, *sizes, 256) == launches
    assert gpusq.lib().gpusq_patch_embed_int8_launches(gpusq.I8, *sizes, 256) == 0
    # fp32 images of 4 GiB or more
    assert gpusq.lib().gpusq_patch_embed_int8_launches(gpusq.F16, 1, 3, 19600, 19600, 14, 640, 768, 1, 256) == 2
    assert gpusq.lib().gpusq_patch_embed_int8_launches(gpusq.F32, 1, 3, 19600, 19600, 14, 640, 768, 1, 256) == 4


# 16 x 16 patches of four channels, timed slower on the kernel for whole rows beyond 512 patches or 160 K outputs, and neighbours that were timed faster
@pytest.mark.parametrize("sizes,launches", [
    ((3, 4, 208, 144, 16, 1024, 648, 1), 4), ((6, 4, 128, 112, 16, 1024, 768, 1), 4), ((2, 4, 368, 320, 16, 1024, 204, 1), 4), ((6, 4, 208, 144, 16, 1024, 200, 1), 4),
    ((6, 3, 128, 112, 16, 768, 768, 1), 2), ((8, 4, 48, 240, 16, 1024, 372, 1), 2), ((6, 4, 32, 144, 16, 1024, 1152, 1), 2)])
def test_few_patches_timed_slower_on_whole_rows_are_four_launches(sizes, launches):
    from paper_2305_10727_amd import gpusq
    assert all(gpusq.lib().gpusq_patch_embed_int8_launches(dt, *sizes, 256) == launches for dt in (gpusq.F32, gpusq.F16))


# sizes that were timed slower behind the range pass, and neighbours that were timed faster: both types, or (fp32, fp16)
@pytest.mark.parametrize("sizes,launches", [
    ((3, 320, 8, 14, 2, 1280, 64, 1), 4), ((5, 64, 64, 72, 4, 1024, 128, 1), 4), ((1, 4, 420, 420, 14, 896, 832, 1), 4), ((1, 3, 420, 420, 14, 640, 576, 1), 2),  # channels
    ((30, 3, 320, 320, 8, 256, 256, 1), 4), ((30, 1, 320, 320, 8, 128, 256, 1), (4, 2)), ((4, 3, 320, 320, 8, 256, 256, 1), 2),  # 8 rows: many patches, few
    ((30, 3, 200, 200, 4, 128, 192, 1), 4), ((30, 2, 200, 200, 4, 128, 192, 1), (4, 2)), ((2, 3, 200, 200, 4, 128, 192, 1), 2),
    ((10, 3, 80, 80, 8, 256, 960, 1), (4, 2)),                                                                                   # few patches for the weights
    ((64, 3, 224, 224, 14, 640, 1472, 1), 4),                                                                                    # channels out
    ((53, 3, 250, 250, 10, 384, 1088, 1), 4), ((51, 3, 250, 250, 10, 384, 1088, 1), 2), ((66, 3, 250, 250, 10, 384, 1088, 1), 2),  # just past a round, in it, beyond
    ((130, 3, 224, 224, 14, 640, 1088, 1), 2)])                                                                                  # (14 rows: there as well)
def test_int8_patch_embeddings_timed_slower_behind_the_range_pass_are_four(sizes, launches):
    from paper_2305_10727_amd import gpusq
    both = launches if isinstance(launches, tuple) else (launches, launches)
    assert tuple(gpusq.lib().gpusq_patch_embed_int8_launches(dt, *sizes, 256) for dt in (gpusq.F32, gpusq.F16)) == both


def test_patch_embedding_argument_checks(lib):
    ERR_NULL, ERR_SHAPE, ERR_ALIGN, ERR_UNSUPPORTED = 1, 2, 3, 4
    vp, i64, ci = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int
    lib.gpusq_patch_embed_fp16.argtypes = [vp] * 5 + [i64] * 7 + [ci, vp]
    call = lambda img=16, W=16, bias=16, Y=16, X=16, B=1, C=3, H=28, Wd=28, P=14, K_pad=592, D=64, epi=1: lib.gpusq_patch_embed_fp16(
        img, W, bias, Y, X, B, C, H, Wd, P, K_pad, D, epi, None)
    for missing in ("img", "W", "bias", "Y", "X"):
        assert call(**{missing: None}) == ERR_NULL
        assert call(**{missing: 24}) == ERR_ALIGN
    for wrong in (dict(B=0), dict(H=27), dict(Wd=30), dict(P=0), dict(K_pad=576), dict(D=0), dict(C=70000)):
        assert call(**wrong) == ERR_SHAPE
    for wrong in (dict(epi=4), dict(K_pad=596), dict(D=66)):
        assert call(**wrong) == ERR_UNSUPPORTED
    lib.gpusq_patch_embed_int8.argtypes = [vp, ci] + [vp] * 8 + [i64] * 7 + [ci, vp]
    call8 = lambda img=16, dt=1, W=16, sa=16, sw=16, bias=16, Y=16, q=16, X=16, ws=16, B=1, C=3, H=28, Wd=28, P=14, K_pad=592, D=64, epi=1: lib.gpusq_patch_embed_int8(
        img, dt, W, sa, sw, bias, Y, q, X, ws, B, C, H, Wd, P, K_pad, D, epi, None)
    for missing in ("img", "W", "sa", "sw", "bias", "Y", "q", "X", "ws"):
        assert call8(**{missing: None}) == ERR_NULL
        assert missing in ("sa", "sw") or call8(**{missing: 24}) == ERR_ALIGN
    for wrong in (dict(B=0), dict(H=27), dict(P=0), dict(K_pad=576), dict(D=0), dict(H=28 * 1400, Wd=28 * 1400)):
        assert call8(**wrong) == ERR_SHAPE
    for wrong in (dict(epi=4), dict(K_pad=596), dict(D=66), dict(dt=2), dict(dt=3)):
        assert call8(**wrong) == ERR_UNSUPPORTED


def test_patch_embedding_refuses_weight_scales_as_the_product_does(lib):
    """gpusq_patch_embed_int8 reads w_scale by 16 bytes, as gpusq_spgemm_int8: from an address that is not aligned to them neither does"""
    ERR_ALIGN = 3
    vp, i64, ci = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int
    lib.gpusq_spgemm_int8.argtypes = [vp, vp, vp, vp, vp, vp, ci, vp, i64, i64, i64, ci, vp]
    lib.gpusq_patch_embed_int8.argtypes = [vp, ci] + [vp] * 8 + [i64] * 7 + [ci, vp]
    for sw in (20, 24, 28):
        assert lib.gpusq_spgemm_int8(16, 16, 16, sw, 16, 16, 1, None, 4, 64, 592, 1, None) == ERR_ALIGN
        for dt in (0, 1):
            for P, H, K_pad in ((14, 28, 592), (16, 32, 768), (28, 28, 2352)):  # in LDS, on whole rows, apart
                assert lib.gpusq_patch_embed_int8(16, dt, 16, 16, sw, 16, 16, 16, 16, 16, 1, 3, H, H, P, K_pad, 64, 1, None) == ERR_ALIGN


def test_empty_of_the_extension_module_is_torch_empty():
    torch = pytest.importorskip("torch")
    from paper_2305_10727_amd import _fastcall
    like = torch.zeros(3)
    for dtype in (torch.float32, torch.float16, torch.int8, torch.uint8, torch.int32):
        for sizes in ((5,), (0,), (4, 6), (1, 0), (2, 3, 4)):
            t = _fastcall.empty(like, dtype, *sizes)
            ref = torch.empty(sizes, dtype=dtype)
            assert type(t) is torch.Tensor and t.shape == ref.shape and t.dtype == ref.dtype and t.device == ref.device and t.stride() == ref.stride()
            assert not t.requires_grad
    assert _fastcall.empty(torch.nn.Parameter(like), torch.int8, 2).requires_grad is False
    with torch.inference_mode():
        assert _fastcall.empty(like, torch.int8, 2).is_inference()
    with pytest.raises(RuntimeError):
        _fastcall.empty(like, torch.int8, -1)
    for wrong in ((None, torch.int8, 2), (like, "int8", 2), (like, torch.int8), (like, torch.int8, 1, 1, 1, 1, 1), (like, torch.int8, 1.5)):
        with pytest.raises(TypeError):
            _fastcall.empty(*wrong)


def test_calls_take_the_address_of_a_tensor_and_of_what_acts_like_one():
    """A tensor, a parameter, a subclass, an object with data_ptr(), an integer and None, checked and not"""
    import ctypes
    torch = pytest.importorskip("torch")
    from paper_2305_10727_amd import _fastcall
    met = []
    c_function = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_uint64)(lambda p: met.append(p) or 0)
    address = ctypes.cast(c_function, ctypes.c_void_p).value
    unchecked, checked = (_fastcall.FastCall("f", address, sig, True) for sig in ("p", "t"))
    x = torch.zeros((6, 8), dtype=torch.int8)

    class Sub(torch.Tensor):
        pass

    class Acts:
        def data_ptr(self):
            return x.data_ptr()

    for v in (x, x[:3], torch.nn.Parameter(x, requires_grad=False), x.as_subclass(Sub), Acts(), x.data_ptr(), x[1:], x.t(), None):
        unchecked(v)
    assert met == [x.data_ptr()] * 6 + [x.data_ptr() + 8, x.data_ptr(), 0]
    checked(None)
    for v in (x, x.as_subclass(Sub)):  # (not on the GPU)
        with pytest.raises(ValueError):
            checked(v)
    with pytest.raises((TypeError, AttributeError)):
        unchecked("x")
    assert met[9:] == [0]


# few rows and small operands; few rows of large ones; many; beyond 512 channels; no whole 64 channels; few slabs to LDS, one round and more; invalid
@pytest.mark.parametrize("M,D,H,launches", [(197, 192, 768, 1), (197, 512, 2048, 3), (12544, 512, 2048, 1), (12608, 768, 3072, 3), (4000, 208, 832, 3),
                                            (4492, 448, 3584, 1), (17053, 384, 3072, 3), (0, 512, 2048, 0), (16, 24, 96, 0)])
def test_launches_behind_attention(M, D, H, launches):
    from paper_2305_10727_amd import gpusq
    assert gpusq.lib().gpusq_block_mlp_int8_launches(M, D, H, 256) == launches


# sizes that were timed slower in one launch, and neighbours that were timed faster: operands of 448 KB; many rows with a hidden layer of half the row or less
@pytest.mark.parametrize("M,D,H,launches", [(104, 320, 960, 3), (221, 320, 960, 3), (122, 448, 576, 3), (1000, 320, 960, 1), (104, 320, 896, 1), (122, 448, 512, 1),
                                            (53810, 512, 64, 3), (62832, 512, 128, 3), (200000, 512, 256, 3), (200000, 448, 64, 3), (30000, 512, 64, 1), (60000, 448, 128, 1), (60000, 512, 320, 1),
                                            (200000, 384, 128, 1)])
def test_layers_behind_attention_timed_slower_in_one_launch_are_three(M, D, H, launches):
    from paper_2305_10727_amd import gpusq
    assert gpusq.lib().gpusq_block_mlp_int8_launches(M, D, H, 256) == launches


class _Recorder:
    """Stands for the library's calls: which ones, with what arguments"""

    def __init__(self):
        self.met = []

    def __getattr__(self, name):
        return lambda *args: self.met.append((name, args))


@pytest.mark.parametrize("change", [None, "fc2.Xq", "fc2.act_scale", "scales", "proj.epilogue", "fc1.epilogue", "fc2.epilogue", "fc2.out_dtype", "rows", "hidden"])
def test_a_block_honours_its_layers_attributes(monkeypatch, change):
    """proj, fc1 and fc2 are one call where that is what they hold, else the layers' own calls on it"""
    torch = pytest.importorskip("torch")
    from paper_2305_10727_amd import gpusq, pipeline
    calls = _Recorder()
    monkeypatch.setattr(pipeline, "_call", calls)
    M, D, H = 32, 64, 256
    block = pipeline.EncoderBlockLinears(M, D, H, {k: torch.ones(1) for k in ("x", "qkv", "attn", "h", "g")}, device="cpu")
    proj, fc1, fc2 = block.proj, block.fc1, block.fc2
    if change == "fc2.Xq":
        fc2.Xq = fc1.Y.clone()
    elif change == "fc2.act_scale":
        fc2.act_scale = torch.ones(1)
    elif change == "scales":
        block.scales = dict(block.scales, g=torch.ones(1))
    elif change == "fc1.epilogue":
        fc1.epilogue = gpusq.EPI_BIAS
    elif change in ("proj.epilogue", "fc2.epilogue"):
        (proj if change[0] == "p" else fc2).epilogue = 0
    elif change == "fc2.out_dtype":
        fc2.out_dtype = torch.int32
    elif change == "rows":
        proj.M = fc1.M = M - 1
    elif change == "hidden":
        fc2.K = H - 64
    biases = [torch.zeros(n) for n in (3 * D, D, H, D)]
    y = block.forward(torch.zeros((M, D), dtype=torch.float16), biases, lambda qkv, out: None)
    assert y is fc2.Y
    got = calls.met[1:]  # (behind qkv)
    if change is None:
        assert [n for n, _ in got] == ["gpusq_block_mlp_int8"]
        return
    assert [n for n, _ in got] == ["gpusq_spgemm_int8_codes", "gpusq_spgemm_int8", "gpusq_spgemm_int8"]
    dt = gpusq._TORCH_DT
    expected = [(proj.Xq, proj.packed, proj.act_scale, proj.w_scale, biases[1], proj.Y, fc1.Xq, fc1.act_scale, proj.M, D, D, proj.epilogue),
                (fc1.Xq, fc1.packed, fc1.act_scale, fc1.w_scale, biases[2], fc1.Y, dt[torch.int8], block.scales["g"], fc1.M, H, D, fc1.epilogue),
                (fc2.Xq, fc2.packed, fc2.act_scale, fc2.w_scale, biases[3], fc2.Y, dt[fc2.out_dtype], None, fc2.M, D, fc2.K, fc2.epilogue)]
    for (_, a), e in zip(got, expected):
        assert len(a) == len(e) and all(x is y if isinstance(y, torch.Tensor) else x == y for x, y in zip(a, e))


@pytest.mark.parametrize("precision", ["int8", "fp16"])
@pytest.mark.parametrize("change", [None, "out_dtype", "rows", "channels"])
def test_a_patch_embedding_honours_its_layers_attributes(monkeypatch, precision, change):
    torch = pytest.importorskip("torch")
    from paper_2305_10727_amd import gpusq, pipeline
    calls = _Recorder()
    monkeypatch.setattr(pipeline, "_call", calls)
    B, C, H, W, P, D = 2, 3, 28, 28, 14, 64
    embed = pipeline.SparsePatchEmbed(B, C, H, W, P, D, precision, device="cpu")
    lin = embed.linear
    if change == "out_dtype":
        lin.out_dtype = torch.int32
    elif change == "rows":
        lin.M = 4
    elif change == "channels":
        lin.N = 32
    img, bias = torch.zeros((B, C, H, W), dtype=torch.float16), torch.zeros(D)
    assert embed.forward(img, bias) is lin.Y
    names = [n for n, _ in calls.met]
    if change is None or (precision, change) == ("fp16", "out_dtype"):  # (the fp16 product has no other output: either way)
        assert change is not None or names == ["gpusq_patch_embed_" + precision]
        return
    assert names == (["gpusq_quantize_int8"] if precision == "int8" else []) + ["gpusq_im2col_patches", "gpusq_spgemm_" + precision]
    if precision == "int8":
        assert calls.met[-1][1][6:] == (gpusq._TORCH_DT[lin.out_dtype], None, lin.M, lin.N, embed.K_pad, lin.epilogue)
    else:
        assert calls.met[-1][1][4:] == (lin.M, lin.N, embed.K_pad, lin.epilogue)


@pytest.mark.parametrize("M,K,N,takes", [(197, 768, 768, True), (2047, 256, 64, True), (2048, 256, 64, True), (4096, 256, 64, True), (4097, 256, 128, False),
                                         (8192, 256, 64, True), (8193, 256, 64, False), (12608, 768, 768, False), (7029, 1152, 256, False)])
def test_layers_whose_gemm_takes_fp16_activations(M, K, N, takes):
    """Those for which the kernel for few rows quantises, whatever their number of rows, and not those of the kernel for many rows (the call
    that makes one launch of both as well)."""
    torch = pytest.importorskip("torch")
    from paper_2305_10727_amd import gpusq
    from paper_2305_10727_amd.pipeline import SparseLinear
    for out in (torch.float16, torch.int8):
        assert SparseLinear(M, K, N, "int8", out_dtype=out, device="cpu").takes_fp16_input() == takes
    if takes:
        assert gpusq.lib().gpusq_linear_int8_launches(gpusq.F16, M, N, K, gpusq.EPI_BIAS, 1, 256) == 1


@pytest.mark.parametrize("M,K,N,gelu,x_dt,out_dt,own,given", [
    # timed with the kernel for whole rows and without: slower with an own range; with either; faster with either
    (30706, 2256, 256, False, 1, 1, 0, 2), (19429, 3312, 192, False, 1, 1, 0, 2), (20738, 3072, 704, True, 1, 1, 0, 2), (26920, 2672, 64, True, 1, 1, 0, 2),
    (32855, 256, 32, False, 0, 2, 0, 2), (22807, 256, 128, True, 0, 2, 0, 2), (29239, 176, 64, True, 0, 1, 0, 2), (27117, 128, 16, True, 0, 1, 0, 2),
    (11620, 2304, 1056, False, 0, 1, 0, 2), (2154, 3264, 704, True, 0, 1, 0, 2),
    (2085, 3920, 640, False, 1, 1, 0, 0), (2164, 1920, 448, True, 1, 2, 0, 0), (28453, 1600, 1920, True, 1, 1, 0, 0),
    (12544, 768, 768, False, 1, 1, 2, 2), (25216, 3072, 768, False, 1, 1, 2, 2), (14070, 576, 256, False, 1, 1, 2, 2), (7029, 1152, 256, False, 1, 1, 2, 2),
    (56475, 3648, 704, False, 1, 1, 2, 2), (50432, 192, 192, False, 1, 1, 2, 2), (12544, 512, 1536, False, 1, 2, 2, 2), (25686, 384, 128, False, 0, 1, 2, 2),
    (29242, 448, 208, False, 0, 1, 2, 2)])
def test_layers_of_the_kernel_for_whole_rows(lib, M, K, N, gelu, x_dt, out_dt, own, given):
    f = lib.gpusq_linear_int8_quantiser
    f.argtypes = [ctypes.c_int, ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int] * 3
    assert (f(x_dt, out_dt, M, N, K, 3 if gelu else 1, 0, 256), f(x_dt, out_dt, M, N, K, 3 if gelu else 1, 1, 256)) == (own, given)
    if out_dt == 1:
        launches = lib.gpusq_linear_int8_launches
        launches.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int] * 3
        assert launches(x_dt, M, N, K, 3 if gelu else 1, 0, 256) == (3 if own == 0 else 2) and launches(x_dt, M, N, K, 3 if gelu else 1, 1, 256) == (2 if given == 0 else 1)


@pytest.mark.parametrize("M,K,N,own,given", [
    # up to 256 and 512 values; 1024 where there are 2^20 outputs, 768 from 2048 rows on; 2^23 outputs at the most; rows of no whole 16 channels
    (1000, 256, 768, 2, 2), (1000, 272, 768, 2, 0), (1000, 512, 768, 2, 0), (1000, 528, 768, 0, 0), (1024, 528, 1024, 2, 0), (2047, 1024, 528, 2, 0),
    (2047, 1040, 528, 0, 0), (2048, 768, 2048, (0, 2), 0), (2048, 784, 2048, 0, 0), (2048, 256, 4096, 2, 2), (2049, 256, 4096, 0, 0), (2000, 256, 1004, 2, 2), (700, 128, 128, 1, 1)])
@pytest.mark.parametrize("x_dt", [0, 1])
def test_short_layers_of_the_kernel_for_whole_rows(lib, M, K, N, own, given, x_dt):
    f = lib.gpusq_linear_int8_quantiser
    f.argtypes = [ctypes.c_int, ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int] * 3
    own = own[x_dt] if isinstance(own, tuple) else own  # (fp32 X: 2^21 outputs at the most for more than 512 values)
    for out_dt in (1, 2):
        for epilogue in (1, 3):
            assert (f(x_dt, out_dt, M, N, K, epilogue, 0, 256), f(x_dt, out_dt, M, N, K, epilogue, 1, 256)) == (own, given)


def _on_whole_rows(lib, M, K, N, fp32, int8_out, gelu, given):
    f = lib.gpusq_linear_int8_quantiser
    f.argtypes = [ctypes.c_int, ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int] * 3
    return f(0 if fp32 else 1, 2 if int8_out else 1, M, N, K, 3 if gelu else 1, given, 256) == 2


# sizes that were timed slower on the kernel for whole rows, which then quantise apart, and neighbours that were timed faster: (M, K, N, fp32, int8 output, GELU, given scale)
@pytest.mark.parametrize("sizes,whole_rows", [
    ((861, 448, 720, 0, 1, 1, 0), False), ((952, 480, 768, 1, 1, 1, 0), False), ((723, 448, 720, 1, 1, 0, 0), False), ((1254, 384, 784, 1, 0, 0, 0), True),  # a slab of 12 blocks; more outputs
    ((367, 400, 1424, 0, 1, 1, 0), False), ((542, 416, 2048, 0, 0, 0, 0), True), ((128, 400, 4432, 0, 1, 1, 0), False), ((345, 208, 3728, 0, 0, 0, 0), True),  # column blocks; 256 values
    ((3998, 400, 1680, 1, 1, 1, 0), False), ((3939, 320, 1936, 1, 1, 1, 0), False), ((2340, 384, 3136, 1, 0, 1, 0), False), ((3939, 320, 1936, 0, 1, 1, 0), True),  # four slabs of fp32
    ((250, 496, 2724, 0, 0, 0, 0), False), ((1136, 512, 540, 1, 0, 0, 0), False), ((237, 464, 3572, 1, 0, 0, 0), False), ((4087, 272, 1544, 1, 0, 1, 0), False),   # rows stored by four
    ((224, 240, 2948, 0, 0, 1, 1), False), ((408, 128, 1432, 1, 0, 1, 1), False), ((368, 192, 2020, 1, 0, 0, 1), False), ((875, 128, 4204, 0, 0, 0, 0), True), ((806, 80, 924, 1, 0, 0, 1), True)])
def test_short_layers_timed_slower_on_whole_rows_quantise_apart(lib, sizes, whole_rows):
    assert _on_whole_rows(lib, *sizes) == whole_rows


# rows of Y of no whole 16 channels, of layers that the estimates take: timed slower on whole rows, and neighbours timed faster
@pytest.mark.parametrize("sizes,whole_rows", [
    ((43513, 208, 60, 0, 1, 0, 1), False), ((18400, 448, 56, 0, 1, 1, 1), False), ((28812, 144, 40, 0, 0, 1, 1), False), ((25599, 64, 52, 0, 0, 0, 0), True),      # one block of channels
    ((58500, 176, 88, 0, 0, 0, 1), False), ((55151, 128, 72, 0, 1, 1, 1), False), ((64607, 80, 124, 1, 0, 1, 0), False),                                          # two
    ((39060, 64, 1080, 0, 1, 0, 0), False), ((29916, 128, 1176, 1, 1, 0, 1), False), ((29308, 160, 696, 1, 1, 0, 0), False), ((16695, 288, 1416, 0, 0, 0, 0), True),  # int8 output of many channels
    ((9464, 384, 124, 1, 1, 0, 0), False), ((7352, 80, 856, 0, 1, 0, 1), True), ((53665, 2288, 748, 0, 0, 1, 1), True), ((7070, 448, 364, 1, 1, 0, 1), True)])
def test_narrow_rows_timed_slower_on_whole_rows_quantise_apart(lib, sizes, whole_rows):
    assert _on_whole_rows(lib, *sizes) == whole_rows


def test_what_quantises_a_layer(lib):
    """The answers of gpusq_linear_int8_quantiser and gpusq_linear_int8_launches agree; int32 output has no kernel for whole rows"""
    f = lib.gpusq_linear_int8_quantiser
    f.argtypes = [ctypes.c_int, ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int] * 3
    launches = lib.gpusq_linear_int8_launches
    launches.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int] * 3
    F32, F16, I8, I32 = range(4)
    for x_dt in (F32, F16):
        for M, N, K, what in ((197, 768, 768, 1), (1576, 1152, 384, 0), (12608, 768, 768, 2), (12608, 3072, 768, 0)):
            assert f(x_dt, F16, M, N, K, 1, 1, 256) == what
            assert launches(x_dt, M, N, K, 1, 1, 256) == (2 if what == 0 else 1)
        assert f(x_dt, I32, 12608, 768, 768, 1, 1, 256) == 0 and f(x_dt, I8, 12608, 768, 768, 1, 1, 256) == 2
    assert f(I8, F16, 197, 768, 768, 0, 1, 256) == f(F16, F32, 197, 768, 768, 0, 1, 256) == f(F16, F16, 197, 768, 100, 0, 1, 256) == f(F16, F16, 0, 768, 768, 0, 1, 256) == -1
