"""One linear layer's full path with preallocated device buffers: prune -> quantise -> compress -> pack (weight
side), quantise activations, sparse GEMM with fused epilogue.  Every step is one call into libgpusq; this class only owns
the buffers and passes pointers (PyTorch = device memory + current stream).  What the caller hands in (weights, activations,
biases, scales) has to be contiguous, on the GPU and of the object's sizes and types: it is not checked here.
"""
import ctypes

import torch

from . import gpusq as G

_call = G.calls_unchecked
_BIAS_GELU = G.EPI_BIAS | G.EPI_GELU


def _p(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


class SparseLinear:
    """Buffers and call sequence for Y = act(X W^T + b) with 2:4-pruned W [N,K].

    precision 'int8': per-output-channel int8 weights, per-tensor int8 activations, int32 accumulation.
    precision 'fp16': fp16 weights and activations, fp32 accumulation.
    x_dtype: dtype of the activations handed in (fp16, or fp32 for the int8 path)."""

    def __init__(self, M, K, N, precision="int8", gelu=False, bias=True, out_dtype=torch.float16, x_dtype=torch.float16,
                 device="cuda"):
        assert precision in ("int8", "fp16")
        self.M, self.K, self.N, self.precision, self.gelu = M, K, N, precision, gelu
        self.out_dtype = out_dtype if precision == "int8" else torch.float16
        e = lambda shape, dt: torch.empty(shape, dtype=dt, device=device)
        self.W_pruned = e((N, K), torch.float32)
        self.epilogue = (G.EPI_BIAS if bias else 0) | (G.EPI_GELU if gelu else 0)
        wdt = torch.int8 if precision == "int8" else torch.float16
        self.W_low = e((N, K), wdt)  # quantised (int8) or rounded (fp16) masked weights: also the dense twin's operand
        self.values = e((N, K // 2), wdt)
        self.meta = e((N, G.meta_row_bytes(K)), torch.uint8)
        self.packed = e((G.packed_bytes(wdt, N, K),), torch.uint8)
        self.Y = e((M, N), self.out_dtype)
        if precision == "int8":
            self.w_scale = e((N,), torch.float32)
            self.act_scale = e((1,), torch.float32)
            self.Xq = e((M, K), torch.int8)
            self.workspace = e((max(G.lib().gpusq_quantize_workspace_bytes(G.PER_TENSOR, M, K), 16),), torch.uint8)
        self.x_dtype = x_dtype

    # ---- weight side (a1, a2, a3 + packing) -------------------------------------------------------------------
    def prepare_weights(self, W, fused=True, intermediates=True):
        """fused=True: one launch (gpusq_prepare_weights); fused=False: the four separate calls.
        intermediates=False (fused only): the pruned fp32 weights, the masked low-precision weights, the canonical values
        and metadata stay in the kernel's registers; only what the sparse GEMM reads (packed operand, scales) is written."""
        N, K = self.N, self.K
        if fused and K * 4 <= 64 * 1024:
            keep = (lambda t: t) if intermediates else (lambda t: None)
            _call.gpusq_prepare_weights(W, G.I8 if self.precision == "int8" else G.F16, keep(self.W_pruned), keep(self.W_low),
                                        self.w_scale if self.precision == "int8" else None, keep(self.values), keep(self.meta),
                                        self.packed, N, K)
            return
        _call.gpusq_prune_2to4(W, self.W_pruned, None, G.F32, N, K)
        if self.precision == "int8":
            _call.gpusq_quantize_int8(self.W_pruned, G.F32, self.W_low, self.w_scale, G.PER_ROW, 0, N, K, None)
            dt = G.I8
        else:
            _call.gpusq_cast_f16(self.W_pruned, self.W_low, N * K)
            dt = G.F16
        _call.gpusq_compress(self.W_low, self.values, self.meta, None, dt, N, K)
        _call.gpusq_pack(self.values, self.meta, self.packed, dt, N, K)

    # ---- activation side + GEMM (a4, a5, a6) --------------------------------------------------------------------
    def quantize_activations(self, X, static=False):
        """static=True: act_scale already holds a calibrated scale and is used as it is (one launch, no range pass)"""
        _call.gpusq_quantize_int8(X, G._TORCH_DT[X.dtype], self.Xq, self.act_scale, G.PER_TENSOR, 1 if static else 0, self.M,
                                  self.K, self.workspace)

    def gemm(self, X, bias, out_scale=None):
        M, N, K = self.M, self.N, self.K
        if self.precision == "int8":
            _call.gpusq_spgemm_int8(self.Xq, self.packed, self.act_scale, self.w_scale, bias, self.Y, G._TORCH_DT[self.out_dtype],
                                    out_scale, M, N, K, self.epilogue)
        else:
            _call.gpusq_spgemm_fp16(X, self.packed, bias, self.Y, M, N, K, self.epilogue)
        return self.Y

    def gemm_and_codes(self, following, bias):
        """INT8 path, fp16 output: the product, and its codes as the input of `following` (of K = this layer's N, its act_scale given)"""
        _call.gpusq_spgemm_int8_codes(self.Xq, self.packed, self.act_scale, self.w_scale, bias, self.Y, following.Xq, following.act_scale,
                                      self.M, self.N, self.K, self.epilogue)
        return self.Y

    def takes_fp16_input(self):
        """True when the INT8 GEMM of this layer should quantise fp16 activations itself (static scale): few rows and a K that
        is not too long, as the library's one-call layer decides it (one launch instead of two).  Not where that call takes its
        kernel for many rows: the GEMM alone does not."""
        return self.precision == "int8" and G.lib().gpusq_linear_int8_quantiser(
            G.F16, G._TORCH_DT[self.out_dtype], self.M, self.N, self.K, self.epilogue, 1, 0) == G.QUANTISE_FEW_ROWS

    def gemm_from_f16(self, X, bias, out_scale=None):
        """INT8 path with a static act_scale: quantise + GEMM in one launch (see takes_fp16_input)"""
        _call.gpusq_spgemm_int8_xf16(X, self.packed, self.act_scale, self.w_scale, bias, self.Y, G._TORCH_DT[self.out_dtype],
                                     out_scale, self.M, self.N, self.K, self.epilogue)
        return self.Y

    def gemm_dense(self, X, bias, out_scale=None):
        """the dense twin on the same masked weights"""
        M, N, K = self.M, self.N, self.K
        if self.precision == "int8":
            _call.gpusq_gemm_int8_dense(self.Xq, self.W_low, self.act_scale, self.w_scale, bias, self.Y,
                                        G._TORCH_DT[self.out_dtype], out_scale, M, N, K, self.epilogue)
        else:
            _call.gpusq_gemm_fp16_dense(X, self.W_low, bias, self.Y, M, N, K, self.epilogue)
        return self.Y

    def forward(self, X, bias, out_scale=None, static=False):
        """static=True (INT8 path): act_scale already holds a calibrated scale and is used as it is"""
        if self.precision == "int8":  # quantise and multiply in one call: one to three launches
            _call.gpusq_linear_int8(X, G._TORCH_DT[X.dtype], self.packed, self.act_scale, 1 if static else 0, self.w_scale, bias, self.Y,
                                    G._TORCH_DT[self.out_dtype], out_scale, self.Xq, self.workspace, self.M, self.N, self.K,
                                    self.epilogue)
            return self.Y
        return self.gemm(X, bias, out_scale)

    def full_path(self, W, X, bias, out_scale=None):
        """all steps of the path in order, as one benchmark step times them"""
        self.prepare_weights(W)
        return self.forward(X, bias, out_scale)


class SparsePatchEmbed:
    """Patch embedding (a convolution with kernel = stride = P) on the sparse GEMM: images [B,C,H,W] -> tokens
    [B*(H/P)*(W/P), D].  The weight [D,C,P,P] is flattened to [D, C*P*P] (zero-padded to whole 128-byte K steps) and
    prepared like a linear layer's; an image is (quantised per tensor and) cut into flattened patches by
    gpusq_im2col_patches, then multiplied by gpusq_spgemm_*; with P = 16 (and a problem large enough for the tile kernel)
    gpusq_patch_embed16_* lets the GEMM gather the patches itself (fused=True, the default where it applies: it saves
    the im2col pass, most on the fp16 path, where a patch row is 32 contiguous bytes; a 16-byte piece of an int8 patch
    row touches a cache line of its own, which gives part of the saving back).  Other patches are one call,
    gpusq_patch_embed_fp16 / _int8, which cuts them in LDS where its sizes favour it; X, which holds flattened patches, is then not
    written.  fused=False: the two calls whatever the sizes."""

    def __init__(self, B, C, H, W, P, D, precision="int8", bias=True, device="cuda", fused=None):
        self.shape = (B, C, H, W)
        can_fuse = P == 16 and B * (H // P) * (W // P) * D > 256 * 1024
        self.fused = can_fuse if fused is None else (fused and can_fuse)
        self.one_call = not self.fused and fused is not False
        self.P, self.D, self.precision = P, D, precision
        self.K = C * P * P
        step = 128 if precision == "int8" else 64  # whole 128-byte K steps: the tile kernel's requirement
        self.K_pad = -(-self.K // step) * step
        self.M = B * (H // P) * (W // P)
        self.linear = SparseLinear(self.M, self.K_pad, D, precision, gelu=False, bias=bias, device=device)
        xdt = torch.int8 if precision == "int8" else torch.float16
        self.X = torch.empty((self.M, self.K_pad), dtype=xdt, device=device)
        if precision == "int8":
            n = B * C * H * W
            self.img_q = torch.empty((B, C, H, W), dtype=torch.int8, device=device)
            self.workspace = torch.empty((max(G.lib().gpusq_quantize_workspace_bytes(G.PER_TENSOR, 1, n), 16),), dtype=torch.uint8,
                                         device=device)

    def prepare_weights(self, Wc):
        """Wc [D,C,P,P] fp32"""
        Wflat = torch.zeros((self.D, self.K_pad), dtype=torch.float32, device=Wc.device)
        Wflat[:, :self.K] = Wc.reshape(self.D, self.K)
        self.linear.prepare_weights(Wflat, fused=self.K_pad * 4 <= 64 * 1024)

    def _linear_as_made(self):
        """Whether the layer has the sizes and the output type that this object gave it (else its own call honours what it has now)"""
        lin = self.linear
        return lin.M == self.M and lin.K == self.K_pad and lin.N == self.D and lin.out_dtype is torch.float16

    def forward(self, img, bias):
        """img [B,C,H,W] fp16 (or fp32 on the int8 path)"""
        B, C, H, W = self.shape
        if self.precision == "int8" and self.fused:  # quantiser and product in one call
            lin = self.linear
            _call.gpusq_patch_embed16_images(img, G._TORCH_DT[img.dtype], lin.packed, lin.act_scale, lin.w_scale, bias, lin.Y, self.img_q, self.workspace,
                                             B, C, H, W, self.D, lin.epilogue & G.EPI_BIAS)
            return lin.Y
        one_call = self.one_call and self._linear_as_made()
        if self.precision == "int8" and one_call:
            lin = self.linear
            lin.Xq = self.X
            _call.gpusq_patch_embed_int8(img, G._TORCH_DT[img.dtype], lin.packed, lin.act_scale, lin.w_scale, bias, lin.Y, self.img_q, self.X, self.workspace,
                                         B, C, H, W, self.P, self.K_pad, self.D, lin.epilogue)
            return lin.Y
        if self.precision == "int8":
            _call.gpusq_quantize_int8(img, G._TORCH_DT[img.dtype], self.img_q, self.linear.act_scale, G.PER_TENSOR, 0, 1,
                                      B * C * H * W, self.workspace)
            src, dt = self.img_q, G.I8
        else:
            src, dt = img, G.F16
        if self.fused:
            lin = self.linear
            _call.gpusq_patch_embed16_fp16(src, lin.packed, bias, lin.Y, B, C, H, W, self.D, lin.epilogue & G.EPI_BIAS)
            return lin.Y
        if one_call:
            lin = self.linear
            _call.gpusq_patch_embed_fp16(src, lin.packed, bias, lin.Y, self.X, B, C, H, W, self.P, self.K_pad, self.D, lin.epilogue)
            return lin.Y
        _call.gpusq_im2col_patches(src, self.X, dt, B, C, H, W, self.P, self.K_pad)
        if self.precision == "int8":
            self.linear.Xq = self.X
        return self.linear.gemm(self.X, bias)


class EncoderBlockLinears:
    """The four linear layers of one encoder block (qkv, proj, fc1, fc2) on the INT8 path with static, calibrated
    activation scales, the deployment form with quantise / dequantise nodes around every linear layer: the
    re-quantisation of a layer's output with the next layer's input scale is fused into its epilogue (qkv -> int8,
    fc1 -> GELU -> int8, which fc2 reads directly).  With a norm one block is six launches of the library:
        quantise x, qkv, [attention], proj, [residual + norm], quantise h, fc1 (GELU), fc2;
    without one proj writes fc1's codes beside its fp16 output, which is a launch less, and up to 512 channels proj, fc1 and fc2 are one launch where that
    is ahead (gpusq_block_mlp_int8), two less again.  qkv, and fc1 behind a norm, quantise their fp16 input on the way in where their sizes favour it: a launch
    less for each.
    Attention and the normalisation are not part of the library: `attention(qkv_int8 [M,3D], out_int8 [M,D])` and
    `norm(proj_fp16 [M,D]) -> fp16 [M,D]` are the caller's (stubs in the tests and the report).  capture() records the
    whole sequence into a HIP graph, which takes the host out of the loop.

    scales: dict of 1-element fp32 device tensors: x (block input), qkv (qkv output), attn (attention output),
    h (fc1 input), g (GELU output = fc2 input)."""

    def __init__(self, M, D, hidden, scales, device="cuda"):
        self.M, self.D, self.hidden = M, D, hidden
        self.qkv = SparseLinear(M, D, 3 * D, "int8", out_dtype=torch.int8, device=device)
        self.proj = SparseLinear(M, D, D, "int8", out_dtype=torch.float16, device=device)
        self.fc1 = SparseLinear(M, D, hidden, "int8", gelu=True, out_dtype=torch.int8, device=device)
        self.fc2 = SparseLinear(M, hidden, D, "int8", out_dtype=torch.float16, device=device)
        self.scales = scales
        self.qkv.act_scale = scales["x"]
        self.proj.act_scale = scales["attn"]
        self.fc1.act_scale = scales["h"]
        self.fc2.act_scale = scales["g"]
        self.fc2.Xq = self.fc1.Y  # fc2 reads the codes fc1's epilogue wrote: no pass in between
        # few rows (the latency kernel) in both qkv and fc1: what quantises its fp16 input in its GEMM (qkv, and fc1 behind a norm) writes
        # no codes, which nothing would read, and a block is four launches; otherwise the one-call layer decides for each and writes
        # them.  Without a norm fc1's codes come from proj, whatever this says.
        self.fold_quantise = self.qkv.takes_fp16_input() and self.fc1.takes_fp16_input()
        self.graph = None

    def prepare_weights(self, Wqkv, Wproj, Wfc1, Wfc2):
        for lin, W in ((self.qkv, Wqkv), (self.proj, Wproj), (self.fc1, Wfc1), (self.fc2, Wfc2)):
            lin.prepare_weights(W)

    def _one_call_behind_attention(self):
        """Whether proj, fc1 and fc2 are what gpusq_block_mlp_int8 stands for.  They are this object's attributes, for a caller to change: other
        buffers, scales, sizes or epilogues are honoured by the layers' own calls."""
        proj, fc1, fc2 = self.proj, self.fc1, self.fc2
        M, D, hidden = proj.M, proj.N, fc1.N
        return (fc2.Xq is fc1.Y and fc2.act_scale is self.scales["g"] and proj.epilogue == fc2.epilogue == G.EPI_BIAS and
                fc1.epilogue == _BIAS_GELU and fc1.out_dtype is torch.int8 and fc2.out_dtype is torch.float16 and
                M == fc1.M == fc2.M and D == proj.K == fc1.K == fc2.N and hidden == fc2.K)

    def forward(self, x, biases, attention, norm=None):
        """x fp16 [M,D]; biases: (b_qkv, b_proj, b_fc1, b_fc2); returns fc2's fp16 output [M,D] (a buffer of this object)"""
        if self.fold_quantise:
            self.qkv.gemm_from_f16(x, biases[0], self.scales["qkv"])
        else:
            self.qkv.forward(x, biases[0], self.scales["qkv"], static=True)
        attention(self.qkv.Y, self.proj.Xq)
        if norm is None:
            proj, fc1, fc2 = self.proj, self.fc1, self.fc2
            if self._one_call_behind_attention():
                _call.gpusq_block_mlp_int8(proj.Xq, proj.packed, proj.act_scale, proj.w_scale, biases[1], proj.Y, fc1.Xq, fc1.act_scale,
                                           fc1.packed, fc1.w_scale, biases[2], fc1.Y, self.scales["g"], fc2.packed, fc2.w_scale, biases[3], fc2.Y,
                                           proj.M, proj.N, fc1.N)
                return fc2.Y
            proj.gemm_and_codes(fc1, biases[1])
            fc1.gemm(None, biases[2], self.scales["g"])
            return fc2.gemm(None, biases[3])
        h = norm(self.proj.gemm(None, biases[1]))
        if self.fold_quantise:
            self.fc1.gemm_from_f16(h, biases[2], self.scales["g"])
        else:
            self.fc1.forward(h, biases[2], self.scales["g"], static=True)
        return self.fc2.gemm(None, biases[3])

    def capture(self, x, biases, attention, norm=None):
        """Records forward() on these buffers into a HIP graph (after one eager run that loads every kernel); replay()
        then reruns it on whatever x and the biases hold at that time."""
        self.forward(x, biases, attention, norm)
        torch.cuda.synchronize()
        self.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self.graph):
            self.forward(x, biases, attention, norm)
        return self.graph

    def replay(self):
        self.graph.replay()
        return self.fc2.Y
