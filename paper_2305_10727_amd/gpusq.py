"""Thin binding over libgpusq.so (include/gpusq.h).  Argument marshalling only: every step of the path runs in the library's
HIP kernels.  PyTorch supplies device memory (`torch.empty`) and the current HIP stream.  The calls that launch kernels go
through the extension module _fastcall (csrc/fastcall.cpp), which converts arguments at a fraction of ctypes' cost; `lib()`
is the ctypes handle on the same library for everything else.

There is no fallback: if the library has not been built, or no GPU tensor is passed, the calls raise.
"""
import ctypes
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libgpusq.so")

OK, ERR_NULL, ERR_SHAPE, ERR_ALIGN, ERR_UNSUPPORTED, ERR_HIP = range(6)
F32, F16, I8, I32 = range(4)
EPI_NONE, EPI_BIAS, EPI_GELU = 0, 1, 2
PER_ROW, PER_TENSOR = 0, 1
QUANTISE_APART, QUANTISE_FEW_ROWS, QUANTISE_WHOLE_ROWS = range(3)

_TORCH_DT = {torch.float32: F32, torch.float16: F16, torch.int8: I8, torch.int32: I32}
_DT_TORCH = {v: k for k, v in _TORCH_DT.items()}

EXPORTS = [
    "gpusq_status_string", "gpusq_last_hip_error", "gpusq_version", "gpusq_prune_2to4", "gpusq_cast_f16",
    "gpusq_quantize_workspace_bytes",
    "gpusq_quantize_int8", "gpusq_compress", "gpusq_check_2to4", "gpusq_decompress", "gpusq_packed_bytes", "gpusq_pack", "gpusq_prepare_weights", "gpusq_spgemm_fp16",
    "gpusq_spgemm_int8", "gpusq_spgemm_int8_codes", "gpusq_spgemm_int8_xf16", "gpusq_spgemm_plan", "gpusq_im2col_patches", "gpusq_patch_embed16_int8", "gpusq_patch_embed16_fp16", "gpusq_patch_embed16_images", "gpusq_patch_embed_fp16", "gpusq_patch_embed_fp16_launches",
    "gpusq_patch_embed_int8", "gpusq_patch_embed_int8_launches", "gpusq_gemm_fp16_dense", "gpusq_gemm_int8_dense",
    "gpusq_prune_4to8_pairs", "gpusq_quantize_rows_int4", "gpusq_compress_int4", "gpusq_decompress_int4",
    "gpusq_int4_to_sparse_int8", "gpusq_prune_n_of_m", "gpusq_force_kernel",
    "gpusq_quantize_tensor_int8_noalloc", "gpusq_linear_int8", "gpusq_linear_int8_launches", "gpusq_linear_int8_quantiser",
    "gpusq_block_mlp_int8", "gpusq_block_mlp_int8_launches",
]


class GpusqError(RuntimeError):
    def __init__(self, status, where):
        self.status = status
        msg = lib().gpusq_status_string(status).decode()
        if status == ERR_HIP:
            msg += " [hip error %d]" % lib().gpusq_last_hip_error()
        super().__init__("%s: %s" % (where, msg))


# C parameters of the calls that launch kernels (fastcall.cpp: p pointer, t checked tensor, i integer, s the stream)
_SIGNATURES = {
    "gpusq_prune_2to4": "tttiiis", "gpusq_cast_f16": "ttis", "gpusq_quantize_int8": "tittiiiits",
    "gpusq_quantize_tensor_int8_noalloc": "tittiiis", "gpusq_compress": "ttttiiis", "gpusq_check_2to4": "titiis",
    "gpusq_decompress": "tttiiis", "gpusq_pack": "tttiiis", "gpusq_prepare_weights": "tittttttiis",
    "gpusq_spgemm_fp16": "ttttiiiis", "gpusq_spgemm_int8": "ttttttitiiiis", "gpusq_spgemm_int8_xf16": "ttttttitiiiis",
    "gpusq_spgemm_int8_codes": "ttttttttiiiis",
    "gpusq_linear_int8": "tittitttitttiiiis",
    "gpusq_block_mlp_int8": "tttttttttttttttttiiis",
    "gpusq_im2col_patches": "ttiiiiiiis", "gpusq_patch_embed16_int8": "ttttttiiiiiis", "gpusq_patch_embed16_fp16": "ttttiiiiiis",
    "gpusq_patch_embed16_images": "titttttttiiiiiis", "gpusq_patch_embed_fp16": "tttttiiiiiiiis",
    "gpusq_patch_embed_int8": "tittttttttiiiiiiiis",
    "gpusq_gemm_fp16_dense": "ttttiiiis", "gpusq_gemm_int8_dense": "ttttttitiiiis", "gpusq_prune_4to8_pairs": "tttiiis",
    "gpusq_quantize_rows_int4": "tittiiis", "gpusq_compress_int4": "ttttiis", "gpusq_decompress_int4": "tttiis",
    "gpusq_int4_to_sparse_int8": "tttttiis", "gpusq_prune_n_of_m": "ttiiiis",
}


class _Calls:
    """The library's launching calls as attributes, built on first use: calls.gpusq_pack(values, meta, packed, dt, N, K) takes
    tensors (or None), checks them (device, contiguity) and raises GpusqError for a status other than OK.  check=False: the
    addresses are passed on as they are; pipeline.py, whose caller answers for the device, the layout and the sizes of what it hands in."""

    def __init__(self, check):
        self._check = check

    def __getattr__(self, name):
        if name not in _SIGNATURES:
            raise AttributeError(name)
        L = lib()
        from . import _fastcall
        _fastcall.setup(torch._C._cuda_getDevice, _stream_of, _raise)
        for n, sig in _SIGNATURES.items():
            assert len(sig) == len(getattr(L, n).argtypes), n
            address = ctypes.cast(getattr(L, n), ctypes.c_void_p).value
            setattr(self, n, _fastcall.FastCall(n, address, sig if self._check else sig.replace("t", "p"), n == "gpusq_check_2to4"))
        return self.__dict__[name]


calls, calls_unchecked = _Calls(True), _Calls(False)


def _raise(status, where):
    raise GpusqError(status, where)


def _stream_of(device):
    return torch.cuda.current_stream(device).cuda_stream


# torch's current stream as a raw hipStream_t.  The public route (torch.cuda.current_stream().cuda_stream) builds a Stream
# object per call and takes about 2.7 us, as long as the launch itself; torch's own raw accessor takes a tenth of that.  It is
# looked up once; without it the public route is used.
_stream_of = getattr(torch._C, "_cuda_getCurrentRawStream", _stream_of)

def _empty(like, dtype, *sizes):
    """torch.empty(sizes, dtype=dtype, device=like.device) at 0.7 us where that takes 1.8; the extension module, loaded on first use, takes its place"""
    global _empty
    from . import _fastcall
    _empty = _fastcall.empty
    return _empty(like, dtype, *sizes)


_lib = None


def lib():
    """Loads libgpusq.so (built by `python -m paper_2305_10727_amd.build`); raises if it is missing."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError("libgpusq.so is not built: run `python -m paper_2305_10727_amd.build` (needs hipcc)")
        L = ctypes.CDLL(LIB_PATH)
        vp, i64, ci = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int
        L.gpusq_status_string.restype = ctypes.c_char_p
        L.gpusq_status_string.argtypes = [ci]
        L.gpusq_last_hip_error.restype = ci
        L.gpusq_version.restype = ci
        L.gpusq_prune_2to4.argtypes = [vp, vp, vp, ci, i64, i64, vp]
        L.gpusq_cast_f16.argtypes = [vp, vp, i64, vp]
        L.gpusq_quantize_workspace_bytes.restype = ctypes.c_size_t
        L.gpusq_quantize_workspace_bytes.argtypes = [ci, i64, i64]
        L.gpusq_quantize_int8.argtypes = [vp, ci, vp, vp, ci, ci, i64, i64, vp, vp]
        L.gpusq_quantize_tensor_int8_noalloc.argtypes = [vp, ci, vp, vp, ci, i64, i64, vp]
        L.gpusq_quantize_tensor_int8_noalloc.restype = ci
        L.gpusq_compress.argtypes = [vp, vp, vp, vp, ci, i64, i64, vp]
        L.gpusq_check_2to4.argtypes = [vp, ci, vp, i64, i64, vp]
        L.gpusq_check_2to4.restype = ci
        L.gpusq_decompress.argtypes = [vp, vp, vp, ci, i64, i64, vp]
        L.gpusq_packed_bytes.restype = ctypes.c_size_t
        L.gpusq_packed_bytes.argtypes = [ci, i64, i64]
        L.gpusq_pack.argtypes = [vp, vp, vp, ci, i64, i64, vp]
        L.gpusq_prepare_weights.argtypes = [vp, ci, vp, vp, vp, vp, vp, vp, i64, i64, vp]
        L.gpusq_prepare_weights.restype = ci
        L.gpusq_spgemm_fp16.argtypes = [vp, vp, vp, vp, i64, i64, i64, ci, vp]
        L.gpusq_spgemm_int8.argtypes = [vp, vp, vp, vp, vp, vp, ci, vp, i64, i64, i64, ci, vp]
        L.gpusq_spgemm_int8_xf16.argtypes = [vp, vp, vp, vp, vp, vp, ci, vp, i64, i64, i64, ci, vp]
        L.gpusq_spgemm_int8_xf16.restype = ci
        L.gpusq_spgemm_int8_codes.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, i64, i64, i64, ci, vp]
        L.gpusq_spgemm_int8_codes.restype = ci
        L.gpusq_block_mlp_int8.argtypes = [vp] * 17 + [i64] * 3 + [vp]
        L.gpusq_block_mlp_int8.restype = ci
        L.gpusq_block_mlp_int8_launches.argtypes = [i64, i64, i64, ci]
        L.gpusq_block_mlp_int8_launches.restype = ci
        L.gpusq_linear_int8.argtypes = [vp, ci, vp, vp, ci, vp, vp, vp, ci, vp, vp, vp, i64, i64, i64, ci, vp]
        L.gpusq_linear_int8.restype = ci
        L.gpusq_linear_int8_launches.argtypes = [ci, i64, i64, i64, ci, ci, ci]
        L.gpusq_linear_int8_launches.restype = ci
        L.gpusq_linear_int8_quantiser.argtypes = [ci, ci, i64, i64, i64, ci, ci, ci]
        L.gpusq_linear_int8_quantiser.restype = ci
        L.gpusq_gemm_fp16_dense.argtypes = [vp, vp, vp, vp, i64, i64, i64, ci, vp]
        L.gpusq_gemm_int8_dense.argtypes = [vp, vp, vp, vp, vp, vp, ci, vp, i64, i64, i64, ci, vp]
        L.gpusq_im2col_patches.argtypes = [vp, vp, ci, i64, i64, i64, i64, i64, i64, vp]
        L.gpusq_patch_embed16_int8.argtypes = [vp, vp, vp, vp, vp, vp, i64, i64, i64, i64, i64, ci, vp]
        L.gpusq_patch_embed16_fp16.argtypes = [vp, vp, vp, vp, i64, i64, i64, i64, i64, ci, vp]
        L.gpusq_patch_embed16_images.argtypes = [vp, ci, vp, vp, vp, vp, vp, vp, vp, i64, i64, i64, i64, i64, ci, vp]
        L.gpusq_patch_embed16_images.restype = ci
        L.gpusq_patch_embed_int8.argtypes = [vp, ci] + [vp] * 8 + [i64] * 7 + [ci, vp]
        L.gpusq_patch_embed_int8.restype = ci
        L.gpusq_patch_embed_int8_launches.argtypes = [ci] + [i64] * 7 + [ci, ci]
        L.gpusq_patch_embed_int8_launches.restype = ci
        L.gpusq_patch_embed_fp16.argtypes = [vp] * 5 + [i64] * 7 + [ci, vp]
        L.gpusq_patch_embed_fp16.restype = ci
        L.gpusq_patch_embed_fp16_launches.argtypes = [i64] * 7 + [ci, ci]
        L.gpusq_patch_embed_fp16_launches.restype = ci
        L.gpusq_spgemm_plan.argtypes = [ci, i64, i64, i64, ci, ci, ctypes.POINTER(ctypes.c_int32)]
        L.gpusq_force_kernel.argtypes = [ci]
        L.gpusq_force_kernel.restype = ci
        L.gpusq_prune_4to8_pairs.argtypes = [vp, vp, vp, ci, i64, i64, vp]
        L.gpusq_prune_n_of_m.argtypes = [vp, vp, ci, ci, i64, i64, vp]
        L.gpusq_int4_to_sparse_int8.argtypes = [vp, vp, vp, vp, vp, i64, i64, vp]
        L.gpusq_quantize_rows_int4.argtypes = [vp, ci, vp, vp, ci, i64, i64, vp]
        L.gpusq_compress_int4.argtypes = [vp, vp, vp, vp, i64, i64, vp]
        L.gpusq_decompress_int4.argtypes = [vp, vp, vp, i64, i64, vp]
        for name in ("gpusq_prune_2to4", "gpusq_cast_f16", "gpusq_quantize_int8", "gpusq_compress", "gpusq_check_2to4", "gpusq_decompress", "gpusq_pack",
                     "gpusq_spgemm_fp16", "gpusq_spgemm_int8", "gpusq_gemm_fp16_dense", "gpusq_gemm_int8_dense"):
            getattr(L, name).restype = ci
        _lib = L
    return _lib


def _ptr(t):
    if t is None:
        return None
    if not t.is_cuda:
        raise ValueError("gpusq works on device tensors only")
    if not t.is_contiguous():
        raise ValueError("gpusq needs contiguous tensors")
    return ctypes.c_void_p(t.data_ptr())


def _stream():
    return ctypes.c_void_p(_stream_of(torch.cuda.current_device()))


def _check(status, where):
    if status != OK:
        raise GpusqError(status, where)


def meta_row_bytes(K):
    return (K // 4 + 1) // 2


def version():
    return lib().gpusq_version()


def prune_2to4(W, out=None, want_mask=False):
    """gpusq_prune_2to4: W [N,K] fp32/fp16 -> pruned W (and the [N,K/4] keep-mask bytes if asked)."""
    N, K = W.shape
    out = _empty(W, W.dtype, N, K) if out is None else out
    mask = _empty(W, torch.uint8, N, max(K // 4, 1)) if want_mask else None
    calls.gpusq_prune_2to4(W, out, mask, _TORCH_DT[W.dtype], N, K)
    return (out, mask) if want_mask else out


def cast_f16(X, out=None):
    """gpusq_cast_f16: fp32 tensor -> fp16 tensor of the same shape (round-to-nearest-even)."""
    out = torch.empty(X.shape, dtype=torch.float16, device=X.device) if out is None else out
    calls.gpusq_cast_f16(X, out, X.numel())
    return out


def quantize_int8(X, mode, scale=None):
    """gpusq_quantize_int8: returns (Xq int8, scale tensor).  mode PER_ROW: scale [rows]; PER_TENSOR: scale [1].
    Pass `scale` (device fp32 tensor) to quantise with given scales."""
    rows, cols = X.shape
    Xq = _empty(X, torch.int8, rows, cols)
    given = scale is not None
    if not given:
        scale = _empty(X, torch.float32, rows if mode == PER_ROW else 1)
    ws_bytes = lib().gpusq_quantize_workspace_bytes(mode, rows, cols)
    ws = _empty(X, torch.uint8, max(ws_bytes, 16))
    calls.gpusq_quantize_int8(X, _TORCH_DT[X.dtype], Xq, scale, mode, int(given), rows, cols, ws)
    return Xq, scale


def quantize_tensor_int8_noalloc(X, Xq, scale, scale_is_input=False):
    """gpusq_quantize_tensor_int8_noalloc: per-tensor codes into the caller's Xq [rows, cols] int8 and scale [1] fp32;
    nothing is allocated, here or in the library."""
    rows, cols = X.shape
    calls.gpusq_quantize_tensor_int8_noalloc(X, _TORCH_DT[X.dtype], Xq, scale, int(bool(scale_is_input)), rows, cols)
    return Xq, scale


def compress(W, want_violations=False):
    """gpusq_compress: W [N,K] fp16/int8 -> (values [N,K/2], meta [N,ceil(K/8)] uint8[, violations int32[1]])."""
    N, K = W.shape
    values = _empty(W, W.dtype, N, max(K // 2, 1))
    meta = _empty(W, torch.uint8, N, max(meta_row_bytes(K), 1))
    viol = _empty(W, torch.int32, 1) if want_violations else None
    calls.gpusq_compress(W, values, meta, viol, _TORCH_DT[W.dtype], N, K)
    return (values, meta, viol) if want_violations else (values, meta)


ERR_NOT_2TO4 = 6


def check_2to4(W):
    """gpusq_check_2to4: W [N,K] fp32/fp16/int8 -> (is_2to4, groups with more than two non-zeros); waits for the stream"""
    N, K = W.shape
    viol = _empty(W, torch.int32, 1)
    st = calls.gpusq_check_2to4(W, _TORCH_DT[W.dtype], viol, N, K)
    if st not in (0, ERR_NOT_2TO4):
        _check(st, "gpusq_check_2to4")
    return st == 0, int(viol.item())


def decompress(values, meta, K):
    N = values.shape[0]
    W = _empty(values, values.dtype, N, K)
    calls.gpusq_decompress(values, meta, W, _TORCH_DT[values.dtype], N, K)
    return W


def prune_n_of_m(W, n, m):
    """gpusq_prune_n_of_m: W [N,K] fp32 -> copy with the n largest magnitudes of every m contiguous elements kept"""
    N, K = W.shape
    out = _empty(W, W.dtype, N, K)
    calls.gpusq_prune_n_of_m(W, out, n, m, N, K)
    return out


def prune_4to8_pairs(W, want_mask=False, one_per_group=False):
    """gpusq_prune_4to8_pairs: W [N,K] fp32 -> pruned copy (and the keep mask [N,K/8] uint8)"""
    N, K = W.shape
    out = _empty(W, W.dtype, N, K)
    mask = _empty(W, torch.uint8, N, K // 8) if want_mask else None
    calls.gpusq_prune_4to8_pairs(W, out, mask, int(one_per_group), N, K)
    return (out, mask) if want_mask else out


def int4_to_sparse_int8(values4, meta4, K, want_mismatches=False):
    """gpusq_int4_to_sparse_int8: INT4 pair-wise storage -> (values [N,K/2] int8, meta [N,K/8] uint8[, mismatches int32[1]])"""
    N = values4.shape[0]
    values8 = _empty(values4, torch.int8, N, K // 2)
    meta8 = _empty(values4, torch.uint8, N, K // 8)
    bad = _empty(values4, torch.int32, 1) if want_mismatches else None
    calls.gpusq_int4_to_sparse_int8(values4, meta4, values8, meta8, bad, N, K)
    return (values8, meta8, bad) if want_mismatches else (values8, meta8)


def quantize_rows_int4(X, scale=None):
    """gpusq_quantize_rows_int4: returns (4-bit codes in an int8 tensor, scale [rows])"""
    rows, cols = X.shape
    Xq = _empty(X, torch.int8, rows, cols)
    given = scale is not None
    if not given:
        scale = _empty(X, torch.float32, rows)
    calls.gpusq_quantize_rows_int4(X, _TORCH_DT[X.dtype], Xq, scale, int(given), rows, cols)
    return Xq, scale


def compress_int4(Wq, want_violations=False):
    """gpusq_compress_int4: Wq [N,K] int8 (4-bit codes) -> (values [N,K/4] uint8, meta [N,ceil(K/16)] uint8[, violations])"""
    N, K = Wq.shape
    values = _empty(Wq, torch.uint8, N, K // 4)
    meta = _empty(Wq, torch.uint8, N, (K // 8 + 1) // 2)
    viol = _empty(Wq, torch.int32, 1) if want_violations else None
    calls.gpusq_compress_int4(Wq, values, meta, viol, N, K)
    return (values, meta, viol) if want_violations else (values, meta)


def decompress_int4(values, meta, K):
    N = values.shape[0]
    W = _empty(values, torch.int8, N, K)
    calls.gpusq_decompress_int4(values, meta, W, N, K)
    return W


def im2col_patches(img, P, K_pad=None):
    """gpusq_im2col_patches: img [B,C,H,W] (int8 or fp16) -> flattened patches [B*(H/P)*(W/P), K_pad] (zero-padded columns)"""
    B, C, H, W = img.shape
    K = C * P * P
    K_pad = K if K_pad is None else K_pad
    X = _empty(img, img.dtype, B * (H // P) * (W // P), K_pad)
    calls.gpusq_im2col_patches(img, X, _TORCH_DT[img.dtype], B, C, H, W, P, K_pad)
    return X


def patch_embed16(img, packed, D, act_scale=None, w_scale=None, bias=None):
    """gpusq_patch_embed16_int8 / _fp16: img [B,C,H,W] int8 or fp16 -> tokens [B*(H/16)*(W/16), D] fp16 (patches gathered by the GEMM)"""
    B, C, H, W = img.shape
    Y = _empty(img, torch.float16, B * (H // 16) * (W // 16), D)
    epi = EPI_BIAS if bias is not None else 0
    if img.dtype == torch.int8:
        calls.gpusq_patch_embed16_int8(img, packed, act_scale, w_scale, bias, Y, B, C, H, W, D, epi)
    else:
        calls.gpusq_patch_embed16_fp16(img, packed, bias, Y, B, C, H, W, D, epi)
    return Y


def spgemm_plan(dtype, M, N, K, epilogue=0, cus=0):
    """gpusq_spgemm_plan: the tile decomposition of a sparse GEMM (host-side; no GPU needed when cus > 0)."""
    out = (ctypes.c_int32 * 8)()
    _check(lib().gpusq_spgemm_plan(_TORCH_DT[dtype], M, N, K, epilogue, cus, out), "gpusq_spgemm_plan")
    keys = ("kernel", "unit_rows", "tiles_n", "full_tm", "full_chunks", "tail_tm", "tiles", "workgroups")
    return dict(zip(keys, list(out)))


def force_kernel(kernel):
    """gpusq_force_kernel (testing aid): 0 / 1 / 2 = run the sparse GEMMs on that kernel, None or -1 = size rules.
    Returns the previous setting."""
    return lib().gpusq_force_kernel(-1 if kernel is None else int(kernel))


def packed_bytes(dtype, N, K):
    return lib().gpusq_packed_bytes(_TORCH_DT[dtype], N, K)


def pack(values, meta, K):
    """gpusq_pack: canonical (values, meta) -> opaque kernel-native buffer (uint8 tensor)."""
    N = values.shape[0]
    nbytes = packed_bytes(values.dtype, N, K)
    if nbytes == 0:
        raise GpusqError(ERR_SHAPE, "gpusq_packed_bytes")
    packed = _empty(values, torch.uint8, nbytes)
    calls.gpusq_pack(values, meta, packed, _TORCH_DT[values.dtype], N, K)
    return packed


def prepare_weights(W, dtype, want_intermediates=False):
    """gpusq_prepare_weights: fp32 W [N,K] -> packed buffer (+ w_scale for int8) in one launch.
    With want_intermediates also returns W_pruned, W_low, values, meta."""
    N, K = W.shape
    dt = _TORCH_DT[dtype]
    packed = _empty(W, torch.uint8, packed_bytes(dtype, N, K))
    w_scale = _empty(W, torch.float32, N) if dtype == torch.int8 else None
    Wp = Wl = values = meta = None
    if want_intermediates:
        Wp = torch.empty_like(W)
        Wl = _empty(W, dtype, N, K)
        values = _empty(W, dtype, N, K // 2)
        meta = _empty(W, torch.uint8, N, meta_row_bytes(K))
    calls.gpusq_prepare_weights(W, dt, Wp, Wl, w_scale, values, meta, packed, N, K)
    out = dict(packed=packed, w_scale=w_scale)
    if want_intermediates:
        out.update(W_pruned=Wp, W_low=Wl, values=values, meta=meta)
    return out


def _epi(bias, gelu):
    return (EPI_BIAS if bias is not None else 0) | (EPI_GELU if gelu else 0)


def spgemm_fp16(X, Wpacked, N, bias=None, gelu=False, out=None):
    M, K = X.shape
    Y = _empty(X, torch.float16, M, N) if out is None else out
    calls.gpusq_spgemm_fp16(X, Wpacked, bias, Y, M, N, K, _epi(bias, gelu))
    return Y


def spgemm_int8(Xq, Wpacked, N, act_scale=None, w_scale=None, bias=None, gelu=False, out_dtype=torch.float16,
                out_scale=None, out=None):
    M, K = Xq.shape
    Y = _empty(Xq, out_dtype, M, N) if out is None else out
    calls.gpusq_spgemm_int8(Xq, Wpacked, act_scale, w_scale, bias, Y, _TORCH_DT[out_dtype], out_scale, M, N, K, _epi(bias, gelu))
    return Y


def spgemm_int8_xf16(X, Wpacked, N, act_scale, w_scale, bias=None, gelu=False, out_dtype=torch.float16, out_scale=None,
                     out=None):
    """X fp16 [M,K], quantised inside the GEMM with the static act_scale (small kernels only: raises GpusqError with
    ERR_UNSUPPORTED for problems of whole K steps that are estimated to be faster on a tile kernel)"""
    M, K = X.shape
    Y = _empty(X, out_dtype, M, N) if out is None else out
    calls.gpusq_spgemm_int8_xf16(X, Wpacked, act_scale, w_scale, bias, Y, _TORCH_DT[out_dtype], out_scale, M, N, K, _epi(bias, gelu))
    return Y


def gemm_fp16_dense(X, W, bias=None, gelu=False, out=None):
    M, K = X.shape
    N = W.shape[0]
    Y = _empty(X, torch.float16, M, N) if out is None else out
    calls.gpusq_gemm_fp16_dense(X, W, bias, Y, M, N, K, _epi(bias, gelu))
    return Y


def gemm_int8_dense(Xq, Wq, act_scale=None, w_scale=None, bias=None, gelu=False, out_dtype=torch.float16, out_scale=None,
                    out=None):
    M, K = Xq.shape
    N = Wq.shape[0]
    Y = _empty(Xq, out_dtype, M, N) if out is None else out
    calls.gpusq_gemm_int8_dense(Xq, Wq, act_scale, w_scale, bias, Y, _TORCH_DT[out_dtype], out_scale, M, N, K, _epi(bias, gelu))
    return Y
