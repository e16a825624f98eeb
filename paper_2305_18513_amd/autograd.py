"""torch.autograd wrappers over the C ABI (Alg. 4 and Sec. 4 of the paper).

Each Function runs its forward through the library, keeps only the compressed
form of the activation its backward needs, and skips the weight gradient of a
frozen layer.  Nothing here computes on its own what a kernel of the library
computes; the dense matrix products of the linear layers are the library's for
fp32 operands of sizes at which it is the quicker one, and torch's otherwise.

  GeluFunction       y = GELU(x); caches x in `bits` bits (per-block scales);
                     backward multiplies by GELU'(x^) straight from the cache.
  LayerNormFunction  frozen: caches the `keep_ppm` largest |x~| of the whole
                     tensor with int32 indices, row pointers and rstd; backward
                     is the paper's input-gradient formula on those pairs, and
                     gamma / beta get no gradient.  Active: caches x exactly
                     and returns all three gradients.  With `quant_bits` the
                     cache is instead the block-scaled codes of x written by the
                     forward kernel itself (plus mean and rstd); backward rebuilds
                     x^ in registers, and an active layer's gamma / beta gradients
                     use the dequantised x^.
  SoftmaxFunction    p = softmax(logits) over the last dimension (at most 2048
                     wide); caches the `keep_ppm` largest probabilities of every
                     row with uint16 columns; backward is the derivative of
                     softmax with the restored (sparse) row in place of p.
  SoftmaxMatmulFunction  out = softmax(logits) @ V with the probabilities shared
                     between the two ops as the paper has it: only the kept
                     pairs and V are cached.  Backward: dP = dO @ V^T (dense
                     product, torch's), dV = P^^T @ dO with P^ restored from the
                     pairs, dlogits from the pairs as in SoftmaxFunction.
  SplitHeadsFunction (q, k^T, v) of the attention products from the rows of a QKV
                     projection in one pass, their gradients back in another.
  MatmulFunction     out = a @ b with both operands cached in 8 bits (the paper's
                     placement for MatMul's activations).
  LinearFunction     the freezing rule of Alg. 4: a layer whose weight does not
                     require a gradient (frozen by the scheduler) keeps nothing of
                     its input and returns no weight gradient; an active one keeps
                     its input in `bits` bits and forms the weight gradient from
                     the dequantised input.

All tensors are CUDA tensors (fp32 or bf16 activations; gamma / beta and the
kept standardised values fp32); the kernels run on torch's current stream.
"""
from __future__ import annotations

import torch
from torch.autograd import forward_ad

from . import binding as sf


def _flat(t: torch.Tensor) -> torch.Tensor:
    return t.contiguous().view(-1)


def _quantise(t: torch.Tensor, bits: int, block: int):
    """(codes, scales) of the flattened tensor, block-scaled."""
    f = _flat(t)
    n = f.numel()
    codes = torch.empty(sf.packed_bytes(n, bits), dtype=torch.uint8, device=t.device)
    scales = torch.empty(sf.num_blocks(n, block), dtype=torch.float32, device=t.device)
    sf.quant_pack(f, sf.Q_BLOCK, bits, block, 0, codes, scales)
    return codes, scales


def _dequantise(codes, scales, bits: int, block: int, shape, dtype) -> torch.Tensor:
    out = torch.empty(shape, dtype=dtype, device=codes.device)
    sf.dequant_unpack(codes, scales, sf.Q_BLOCK, bits, block, 0, out.view(-1))
    return out


def _right(t: torch.Tensor) -> torch.Tensor:
    """The right operand of a batched product, laid out for bf16: torch's bf16 product has faulted the GPU where it was a
    transposed view."""
    return t.contiguous() if t.dtype == torch.bfloat16 else t


class MatmulFunction(torch.autograd.Function):
    """out = a @ b with both operands cached in `bits` bits (the paper keeps MatMul's activations in 8 bits);
    backward multiplies the incoming gradient with the dequantised operands."""

    @staticmethod
    def forward(ctx, a: torch.Tensor, b: torch.Tensor, bits: int = 8, block: int = 64):
        out = torch.matmul(a, _right(b))
        ca, sa = _quantise(a, bits, block)
        cb, sb = _quantise(b, bits, block)
        ctx.save_for_backward(ca, sa, cb, sb)
        ctx.meta = (bits, block, a.shape, b.shape, a.dtype)
        return out

    @staticmethod
    def backward(ctx, grad_output: torch.Tensor):
        ca, sa, cb, sb = ctx.saved_tensors
        bits, block, sha, shb, dtype = ctx.meta
        b_hat = _dequantise(cb, sb, bits, block, shb, dtype)
        da = torch.matmul(grad_output, _right(b_hat.transpose(-1, -2)))
        del b_hat
        a_hat = _dequantise(ca, sa, bits, block, sha, dtype)
        db = torch.matmul(a_hat.transpose(-1, -2), _right(grad_output))
        return da, db, None, None


class GeluFunction(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x: torch.Tensor, bits: int = 4, block: int = 64):
        xf = _flat(x)
        n = xf.numel()
        y = torch.empty_like(xf)
        codes = torch.empty(sf.packed_bytes(n, bits), dtype=torch.uint8, device=x.device)
        scales = torch.empty(sf.num_blocks(n, block), dtype=torch.float32, device=x.device)
        sf.gelu_quant_pack(xf, sf.Q_BLOCK, bits, block, 0, y, codes, scales)
        ctx.save_for_backward(codes, scales)
        ctx.quant = (bits, block)
        return y.view(x.shape)

    @staticmethod
    def backward(ctx, grad_output: torch.Tensor):
        codes, scales = ctx.saved_tensors
        bits, block = ctx.quant
        dy = _flat(grad_output)
        dx = torch.empty_like(dy)
        sf.gelu_backward_dequant(codes, scales, sf.Q_BLOCK, bits, block, 0, dy, dx)
        return dx.view(grad_output.shape), None, None


class LayerNormFunction(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x: torch.Tensor, gamma: torch.Tensor, beta: torch.Tensor, eps: float = 1e-5,
                frozen: bool = False, keep_ppm: int = 100000, quant_bits: int = 0, block: int = 64):
        H = x.shape[-1]
        x2 = x.contiguous().view(-1, H)
        rows = x2.shape[0]
        y = torch.empty_like(x2)
        mean = torch.empty(rows, dtype=torch.float32, device=x.device)
        rstd = torch.empty(rows, dtype=torch.float32, device=x.device)
        ctx.frozen = frozen
        ctx.quant = (quant_bits, block)
        if quant_bits:
            n = x2.numel()
            codes = torch.empty(sf.packed_bytes(n, quant_bits), dtype=torch.uint8, device=x.device)
            scales = torch.empty(sf.num_blocks(n, block), dtype=torch.float32, device=x.device)
            sf.layernorm_forward_quant_pack(x2, gamma, beta, eps, quant_bits, block, y, mean, rstd, codes, scales)
            ctx.save_for_backward(codes, scales, mean, rstd, gamma)
            return y.view(x.shape)
        sf.layernorm_forward(x2, gamma, beta, eps, y, mean, rstd)
        if frozen:
            n = x2.numel()
            k = sf.keep_count(n, keep_ppm)
            vals = torch.empty(k, dtype=torch.float32, device=x.device)
            idx = torch.empty(k, dtype=torch.int32, device=x.device)
            row_ptr = torch.empty(rows + 1, dtype=torch.int32, device=x.device)
            if k > 0:
                sf.prune_global_standardized(x2, mean, rstd, k, vals, idx, True, None, row_ptr)
            else:
                row_ptr.zero_()
            ctx.k = k
            ctx.save_for_backward(vals, idx, row_ptr, rstd, gamma)
        else:
            ctx.save_for_backward(x2, mean, rstd, gamma)
        return y.view(x.shape)

    @staticmethod
    def backward(ctx, grad_output: torch.Tensor):
        H = grad_output.shape[-1]
        dy = grad_output.contiguous().view(-1, H)
        none = (None,) * 5
        bits, block = ctx.quant
        if bits:
            codes, scales, mean, rstd, gamma = ctx.saved_tensors
            dx = torch.empty_like(dy)
            sf.layernorm_backward_dequant(codes, scales, bits, block, mean, rstd, gamma, dy, dx)
            if ctx.frozen:
                return (dx.view(grad_output.shape), None, None) + none
            x_hat = torch.empty_like(dy)
            sf.dequant_unpack(codes, scales, sf.Q_BLOCK, bits, block, 0, x_hat.view(-1))
            dgamma, dbeta = torch.empty_like(gamma), torch.empty_like(gamma)
            sf.layernorm_param_grads(x_hat, mean, rstd, dy, dgamma, dbeta)
            return (dx.view(grad_output.shape), dgamma, dbeta) + none
        if ctx.frozen:
            vals, idx, row_ptr, rstd, gamma = ctx.saved_tensors
            dx = torch.empty_like(dy)
            sf.layernorm_backward_pruned(vals, idx, row_ptr, ctx.k, rstd, gamma, dy, dx)
            return (dx.view(grad_output.shape), None, None) + none
        x2, mean, rstd, gamma = ctx.saved_tensors
        dgamma, dbeta = torch.empty_like(gamma), torch.empty_like(gamma)
        sf.layernorm_param_grads(x2, mean, rstd, dy, dgamma, dbeta)
        dx = torch.empty_like(dy)
        sf.layernorm_backward(x2, mean, rstd, gamma, dy, dx)
        return (dx.view(grad_output.shape), dgamma, dbeta) + none


class SoftmaxFunction(torch.autograd.Function):
    @staticmethod
    def forward(ctx, logits: torch.Tensor, keep_ppm: int = 100000):
        cols = logits.shape[-1]
        l2 = logits.contiguous().view(-1, cols)
        rows = l2.shape[0]
        k = max(1, sf.keep_count(cols, keep_ppm))
        probs = torch.empty_like(l2)
        vals = torch.empty(rows, k, dtype=l2.dtype, device=l2.device)
        idx = torch.empty(rows, k, dtype=torch.uint16, device=l2.device)
        sf.softmax_prune(l2, k, probs, vals, idx)
        ctx.save_for_backward(vals, idx)
        return probs.view(logits.shape)

    @staticmethod
    def backward(ctx, grad_output: torch.Tensor):
        vals, idx = ctx.saved_tensors
        cols = grad_output.shape[-1]
        dp = grad_output.contiguous().view(-1, cols)
        ds = torch.empty_like(dp)
        sf.softmax_backward_pruned(vals, idx, None, dp, ds)
        return ds.view(grad_output.shape), None


class SoftmaxMatmulFunction(torch.autograd.Function):
    @staticmethod
    def forward(ctx, logits: torch.Tensor, v: torch.Tensor, keep_ppm: int = 100000, v_bits: int = 0, block: int = 64):
        # logits (..., Tq, Tk), v (..., Tk, D); v_bits != 0 caches V quantised as well
        cols = logits.shape[-1]
        l2 = logits.contiguous().view(-1, cols)
        rows = l2.shape[0]
        k = max(1, sf.keep_count(cols, keep_ppm))
        probs = torch.empty_like(l2)
        vals = torch.empty(rows, k, dtype=l2.dtype, device=l2.device)
        idx = torch.empty(rows, k, dtype=torch.uint16, device=l2.device)
        sf.softmax_prune(l2, k, probs, vals, idx)
        out = torch.matmul(probs.view(logits.shape), _right(v))
        if v_bits:
            cv, sv = _quantise(v, v_bits, block)
            ctx.save_for_backward(vals, idx, cv, sv)
        else:
            ctx.save_for_backward(vals, idx, v)
        ctx.meta = (logits.shape, v.shape, v.dtype, v_bits, block)
        return out

    @staticmethod
    def backward(ctx, grad_output: torch.Tensor):
        shape, v_shape, v_dtype, v_bits, block = ctx.meta
        if v_bits:
            vals, idx, cv, sv = ctx.saved_tensors
            v = _dequantise(cv, sv, v_bits, block, v_shape, v_dtype)
        else:
            vals, idx, v = ctx.saved_tensors
        cols = shape[-1]
        rows = vals.shape[0]
        if grad_output.dim() > 3:                           # (three dimensions are multiplied as they lie)
            grad_output = grad_output.contiguous()          # both products would lay out a transposed one for themselves
        dp = torch.matmul(grad_output, _right(v.transpose(-1, -2))).contiguous().view(rows, cols)
        p_hat = torch.empty(rows, cols, dtype=vals.dtype, device=vals.device)
        sf.restore_scores(vals, idx, None, p_hat)
        dv = torch.matmul(p_hat.view(shape).transpose(-1, -2), _right(grad_output))
        ds = torch.empty_like(dp)
        sf.softmax_backward_pruned(vals, idx, None, dp, ds)
        return ds.view(shape), dv, None, None, None


class SplitHeadsFunction(torch.autograd.Function):
    """(q, k^T, v) of the attention products from the rows (B, T, 3 * H) of a QKV projection, q times ``q_scale``; backward
    lays the three gradients into one row buffer.  Nothing is kept."""

    @staticmethod
    def forward(ctx, qkv: torch.Tensor, heads: int, q_scale: float):
        B, T, H3 = qkv.shape
        D = H3 // (3 * heads)
        q = torch.empty(B, heads, T, D, dtype=qkv.dtype, device=qkv.device)
        kt = torch.empty(B, heads, D, T, dtype=qkv.dtype, device=qkv.device)
        v = torch.empty_like(q)
        sf.split_heads(qkv.contiguous(), q_scale, q, kt, v)
        ctx.meta = (qkv.shape, q_scale)
        return q, kt, v

    @staticmethod
    def backward(ctx, dq: torch.Tensor, dkt: torch.Tensor, dv: torch.Tensor):
        shape, q_scale = ctx.meta
        dqkv = torch.empty(shape, dtype=dq.dtype, device=dq.device)
        sf.merge_heads(dq.contiguous(), dkt.contiguous(), dv.contiguous(), q_scale, dqkv)
        return dqkv, None, None


def _plain(t: torch.Tensor) -> bool:
    """Whether a kernel may be handed the tensor's memory as it is."""
    return (type(t) in (torch.Tensor, torch.nn.Parameter) and torch._C._has_storage(t) and t.is_cuda
            and t.is_contiguous() and not t.is_neg() and not t._is_zerotensor() and t.data_ptr() % 16 == 0)


def _watched() -> bool:
    """Whether more than the value is asked for, or less: a product to be differentiated (either way), cast, traced or
    intercepted, or one for which the program allows torch fewer than 32 bits."""
    return (torch.is_grad_enabled() or torch.is_autocast_enabled() or torch.compiler.is_compiling() or torch.jit.is_tracing()
            or forward_ad._current_level >= 0 or torch._C._len_torch_dispatch_stack() > 0 or torch._C._len_torch_function_stack() > 0
            # torch.backends.cuda.matmul.fp32_precision, which takes 2.1 us to read, this 0.6
            or torch._C._get_fp32_precision_getter("cuda", "matmul") not in ("none", "ieee"))


_MOST_TILES = (1 << 31) // 512                             # of 128 x 64 that a launch of the library's product can have


def _quicker(M: int, N: int, K: int, transposed: bool) -> bool:
    """Whether the library's product takes the shorter time on the GPU (rows x columns x depth, torch's and this in us).

    It does from about 170 tiles of 128 x 64 on, two for three compute units (1792 x 768 x 768 25.2 and 22.0, 3600 x 384 x 384 19.5 and
    13.4, 4096 x 768 x 3072 140 and 102); fewer torch splits along their depth (2048 x 512 x 2048 35 and 50, 1024 x 768 x 768 14 and
    22, 257 x 256 x 256 5.5 and 9.5).  Weights that lie K x N and are deep need 208 (1500 x 960 x 3072 78 and 81, 3300 x 512 x 2048
    57.1 and 56.0), and a quarter of the tiles at most may be padding (260 x 6144 x 1024 32 and 35, 400 x 6000 x 1024 55 and 42).
    Nor do tall ones of few columns and some depth, which go in tiles of 96 columns (40000 x 64 x 1024 54 and 69, 34000 x 128 x 1536 118 and
    139; 22000 x 128 x 1024, whose tiles have 64, 70 and 45), or one step of depth (17000 x 128 x 32 6.7 and 8.7).
    And where torch does not split: up to 256 x 256 and a depth below 1024, but for the very smallest (256 x 256 x 256 63 and 9.5,
    128 x 128 x 768 88 and 21, 64 x 192 x 64 7.1 and 5.9, 64 x 128 x 64 5.5 and 5.9; of depth 1024 8 and 26)."""
    outputs, tiles = M * N, -(-M // 128) * -(-N // 64)
    if M <= 256 and N <= 256 and 64 <= K < 1024:
        return outputs >= 64 * 192
    if K < 64 or (M > 256 * 128 and N <= 128 and K >= 512):
        return False
    return outputs >= (168 if transposed or K <= 1536 else 208) * 128 * 64 and 4 * outputs >= 3 * 128 * 64 * tiles and tiles <= _MOST_TILES


def _dense(x: torch.Tensor, weight: torch.Tensor, transposed: bool):
    """x @ weight.T or x @ weight over x's last dimension by the library's fp32 product, or None where that is torch's."""
    if x.dtype != torch.float32 or weight.dtype != torch.float32 or x.dim() < 2 or weight.dim() != 2:
        return None
    K = x.shape[-1]
    N, depth = weight.shape if transposed else weight.shape[::-1]
    if depth != K or K == 0 or K % 32 != 0:
        return None
    M = x.numel() // K
    if not _quicker(M, N, K, transposed) or _watched() or not (_plain(x) and _plain(weight)):
        return None
    if not (x.get_device() == weight.get_device() == torch.cuda.current_device()):
        return None                                        # the library launches on the current device
    y = torch.empty(*x.shape[:-1], N, dtype=x.dtype, device=x.device)
    sf.product(x.view(M, K), weight, transposed, y.view(M, N))
    return y


class LinearFunction(torch.autograd.Function):
    """y = x W^T (+ b) under the freezing rule of Alg. 4.  Whether the layer is frozen is read off the weight itself
    (``weight.requires_grad``, which is what an inter-layer scheduler flips between iterations): a frozen layer
    keeps nothing of x and produces no weight gradient; an active one keeps x as ``bits``-bit block-scaled codes
    and forms its weight gradient from the dequantised x^.  The library's fp32 product (sizes: ``_quicker``) holds all bits of
    its operands and is no further from the exact one than fp32 additions in any order; where the program allows torch fewer
    bits (``torch.set_float32_matmul_precision``) the products are torch's."""

    @staticmethod
    def forward(ctx, x: torch.Tensor, weight: torch.Tensor, bias, bits: int = 8, block: int = 64):
        y = _dense(x, weight, True) if bias is None else None
        if y is None:
            y = torch.nn.functional.linear(x, weight, bias)
        ctx.cache = None                                   # descriptor of what is kept of x: nothing, or (bits, block, shape, dtype)
        ctx.bias_active = bias is not None and bias.requires_grad
        if weight.requires_grad:
            codes, scales = _quantise(x, bits, block)
            ctx.cache = (bits, block, x.shape, x.dtype)
            ctx.save_for_backward(weight, codes, scales)
        else:
            ctx.save_for_backward(weight)
        return y

    @staticmethod
    def backward(ctx, dy: torch.Tensor):
        weight = ctx.saved_tensors[0]
        dx = None
        if ctx.needs_input_grad[0]:
            dx = _dense(dy, weight, False)
            if dx is None:
                dx = dy.matmul(weight)
        dy2 = dy.reshape(-1, dy.shape[-1])
        dw = None
        if ctx.cache is not None:
            bits, block, shape, dtype = ctx.cache
            x_hat = _dequantise(ctx.saved_tensors[1], ctx.saved_tensors[2], bits, block, shape, dtype)
            dw = dy2.t().mm(x_hat.view(-1, shape[-1]))
        db = dy2.sum(0) if ctx.bias_active else None
        return dx, dw, db, None, None


def _rows_of_vectors(dim: int, t: torch.Tensor) -> bool:
    """Whether a head's elements are whole 16-byte vectors, which is what split_heads and merge_heads move."""
    return dim * t.element_size() % 16 == 0


def _halves(dim: int) -> bool:
    """Whether sqrt(dim) is a power of two."""
    return dim > 0 and dim & (dim - 1) == 0 and dim.bit_length() % 2 == 1


def encoder_block_params(hidden: int, device="cuda", seed: int = 0, dtype=torch.float32):
    """Random weights of one encoder block (QKV, projection, two feed-forward matrices, two LayerNorms)."""
    g = torch.Generator(device=device).manual_seed(seed)

    def mat(rows, cols):
        return torch.nn.Parameter((torch.randn(rows, cols, generator=g, device=device) * 0.03).to(dtype))

    def vec(value):
        return torch.nn.Parameter(torch.full((hidden,), value, device=device))

    return {"wqkv": mat(3 * hidden, hidden), "wo": mat(hidden, hidden), "w1": mat(4 * hidden, hidden),
            "w2": mat(hidden, 4 * hidden), "g1": vec(1.0), "b1": vec(0.0), "g2": vec(1.0), "b2": vec(0.0)}


def frozen_encoder_block(x: torch.Tensor, p: dict, heads: int, wrapped: bool, keep_ppm: int = 100000,
                         gelu_bits: int = 4, block: int = 64) -> torch.Tensor:
    """One pre-LN encoder block whose layers are all frozen: with ``wrapped`` the activations kept
    for the backward pass are the compressed ones (pruned LayerNorm input, pruned attention probabilities shared by
    Softmax and MatMul, 4-bit GELU input, nothing for the frozen linear layers); without, plain torch ops."""
    B, T, H = x.shape
    D = H // heads
    F = torch.nn.functional

    def split(t):
        return t.reshape(B, T, heads, D).transpose(1, 2)

    if wrapped:
        w = {name: t.detach() for name, t in p.items()}    # frozen: the scheduler has switched their gradients off
        h = LayerNormFunction.apply(x, p["g1"], p["b1"], 1e-5, True, keep_ppm)
        qkv = LinearFunction.apply(h, w["wqkv"], None, 8, block)
        if _rows_of_vectors(D, qkv):
            # 1 / sqrt(D) goes onto q where it is a power of two: that commutes with every rounding on the way (entries of q
            # or its gradient below 1e-35 apart, which may become subnormal or leave the 8-bit cache's range), so these are
            # the numbers of the divided products.  Any other divides them.  (32 x 128 x 768, fp32, forward and backward: heads
            # of 32 1442 -> 1383 us, 64 1360 -> 1290, 96 1325 -> 1276, 128 1328 -> 1260.)
            on_q = _halves(D)
            q, kt, v = SplitHeadsFunction.apply(qkv, heads, 1.0 / D ** 0.5 if on_q else 1.0)
            s = MatmulFunction.apply(q, kt, 8, block)
            s = s if on_q else s / D ** 0.5
        else:
            q, k_, v = qkv.chunk(3, dim=-1)
            s = MatmulFunction.apply(split(q).contiguous(), split(k_).transpose(-1, -2).contiguous(), 8, block) / D ** 0.5
            v = split(v).contiguous()
        a = SoftmaxMatmulFunction.apply(s, v, keep_ppm, 8, block).transpose(1, 2).reshape(B, T, H)
        y = x + LinearFunction.apply(a, w["wo"], None, 8, block)
        h = LayerNormFunction.apply(y, p["g2"], p["b2"], 1e-5, True, keep_ppm)
        h = LinearFunction.apply(h, w["w1"], None, 8, block)
        h = LinearFunction.apply(GeluFunction.apply(h, gelu_bits, block), w["w2"], None, 8, block)
        return y + h
    h = F.layer_norm(x, (H,), p["g1"].to(x.dtype), p["b1"].to(x.dtype), 1e-5)
    q, k_, v = F.linear(h, p["wqkv"]).chunk(3, dim=-1)
    s = torch.matmul(split(q), split(k_).transpose(-1, -2)) / D ** 0.5
    a = torch.matmul(torch.softmax(s, -1), split(v)).transpose(1, 2).reshape(B, T, H)
    y = x + F.linear(a, p["wo"])
    h = F.layer_norm(y, (H,), p["g2"].to(x.dtype), p["b2"].to(x.dtype), 1e-5)
    h = F.linear(F.gelu(F.linear(h, p["w1"])), p["w2"])
    return y + h


def held_activation_bytes(fn) -> tuple:
    """(bytes that stay allocated between the forward pass of ``fn`` and its backward pass, apart from the output;
    milliseconds of forward + backward)."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.memory_allocated()
    t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    t0.record()
    out = fn()
    torch.cuda.synchronize()
    kept = torch.cuda.memory_allocated() - before - out.numel() * out.element_size()
    out.sum().backward()
    t1.record()
    torch.cuda.synchronize()
    return kept, t0.elapsed_time(t1)
