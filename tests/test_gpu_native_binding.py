"""The native form of the step's calls against the general (ctypes) path: over every form of argument the two give the
same bytes, the same exception or the same status, and what is not plain is left to the general path."""
import numpy as np
import pytest
import torch

from paper_2305_18513_amd import binding as sf
from tests.gpu_util import require_gpu, to_np


def _general(fn, *args, **kwargs):
    """The wrapper with its native form switched off."""
    name = "_native_" + fn.__name__
    fast = getattr(sf, name)
    setattr(sf, name, lambda *a: NotImplemented)
    try:
        return fn(*args, **kwargs)
    finally:
        setattr(sf, name, fast)


def _outcome(call, outputs):
    for t in outputs:
        t.view(torch.uint8).fill_(0x5A)
    try:
        result = call()
    except Exception as e:                                             # noqa: BLE001 - the kind and the text are compared
        return type(e), str(e), getattr(e, "status", None)
    torch.cuda.synchronize()
    return result, [to_np(t).tobytes() for t in outputs]


def _calls(dt):
    """name -> (function, arguments, positions of the outputs among them)"""
    g = torch.Generator(device="cuda").manual_seed(3)
    rows, cols, H, k = 70, 48, 128, 4
    n = rows * H

    def randn(*shape):
        return torch.randn(*shape, generator=g, device="cuda").to(dt)

    def f32(*shape):
        return torch.randn(*shape, generator=g, device="cuda").abs() + 0.5

    def empty(*shape, dtype):
        return torch.empty(*shape, dtype=dtype, device="cuda")

    x, dy = randn(rows, H), randn(rows, H)
    codes, scales = empty(n // 2, dtype=torch.uint8), empty(n // 64, dtype=torch.float32)
    sf.quant_pack(x.view(-1), sf.Q_BLOCK, 4, 64, 0, codes, scales)
    p = torch.softmax(randn(rows, cols).float() * 2, -1).to(dt)
    vals, idx = empty(rows, k, dtype=dt), empty(rows, k, dtype=torch.uint16)
    counts = empty(rows, dtype=torch.int32)
    sf.prune_scores(p, k, sf.PRUNE_TOPK, 0.0, vals, idx, None)
    mean, rstd, gamma = x.float().mean(1), 1 / x.float().std(1), f32(H)
    kg = n // 10
    gv, gi, rp = empty(kg, dtype=torch.float32), empty(kg, dtype=torch.int32), empty(rows + 1, dtype=torch.int32)
    tp = empty(sf.global_tile_ptr_len(n), dtype=torch.int32)
    sf.prune_global_standardized(x, mean, rstd, kg, gv, gi, True, tp, rp)
    ws = empty(sf.prune_global_workspace(n), dtype=torch.uint8)
    y, dx = torch.empty_like(x), torch.empty_like(x)
    d, numel = empty(2, dtype=torch.float32), [1000, 24]
    w_prev, w_cur = [f32(m) for m in numel], [f32(m) for m in numel]
    plan = empty(sf.layer_delta_workspace(numel), dtype=torch.uint8)
    sf.layer_delta_plan(w_prev, w_cur, plan)
    new = lambda t: torch.empty_like(t)                                # noqa: E731
    return {
        "quant_pack": (sf.quant_pack, [x.view(-1), sf.Q_BLOCK, 4, 64, 0, new(codes), new(scales)], (5, 6)),
        "quant_pack_fixed": (sf.quant_pack, [x.view(-1), sf.Q_FIXED, 8, 64, 4, empty(n, dtype=torch.uint8), None], (5,)),
        "dequant_unpack": (sf.dequant_unpack, [codes, scales, sf.Q_BLOCK, 4, 64, 0, y.view(-1)], (6,)),
        "gelu_quant_pack": (sf.gelu_quant_pack, [x.view(-1), sf.Q_BLOCK, 4, 64, 0, new(y).view(-1), new(codes), new(scales)], (5, 6, 7)),
        "gelu_backward_dequant": (sf.gelu_backward_dequant, [codes, scales, sf.Q_BLOCK, 4, 64, 0, dy.view(-1), dx.view(-1)], (7,)),
        "prune_scores": (sf.prune_scores, [p, k, sf.PRUNE_TOPK, 0.0, new(vals), new(idx), None], (4, 5)),
        "prune_scores_threshold": (sf.prune_scores, [p, k, sf.PRUNE_THRESHOLD, 0.05, new(vals), new(idx), counts], (4, 5, 6)),
        "restore_scores": (sf.restore_scores, [vals, idx, None, new(p)], (3,)),
        "softmax_prune": (sf.softmax_prune, [randn(rows, cols), k, new(p), new(vals), new(idx)], (2, 3, 4)),
        "softmax_backward_pruned": (sf.softmax_backward_pruned, [vals, idx, None, randn(rows, cols), new(p)], (4,)),
        "prune_global_standardized": (sf.prune_global_standardized, [x, mean, rstd, kg, new(gv), new(gi), True, new(tp), new(rp), ws],
                                      (4, 5, 7, 8)),
        "prune_global_standardized_own": (sf.prune_global_standardized, [x, mean, rstd, kg, new(gv), new(gi)], (4, 5)),
        "layernorm_forward": (sf.layernorm_forward, [x, gamma, f32(H), 1e-5, y, new(mean), new(rstd)], (4, 5, 6)),
        "layernorm_backward": (sf.layernorm_backward, [x, mean, rstd, gamma, dy, dx], (5,)),
        "layernorm_backward_pruned": (sf.layernorm_backward_pruned, [gv, gi, rp, kg, rstd, gamma, dy, dx], (7,)),
        "layernorm_forward_quant_pack": (sf.layernorm_forward_quant_pack,
                                         [x, gamma, f32(H), 1e-5, 4, 64, y, new(mean), new(rstd), new(codes), new(scales)], (6, 7, 8, 9, 10)),
        "layernorm_backward_dequant": (sf.layernorm_backward_dequant, [codes, scales, 4, 64, mean, rstd, gamma, dy, dx], (8,)),
        "split_heads": (sf.split_heads, [randn(3, 5, 48), 0.25, randn(3, 2, 5, 8), randn(3, 2, 8, 5), randn(3, 2, 5, 8)], (2, 3, 4)),
        "merge_heads": (sf.merge_heads, [randn(3, 2, 5, 8), randn(3, 2, 8, 5), randn(3, 2, 5, 8), 0.25, randn(3, 5, 48)], (4,)),
        "product": (sf.product, [f32(40, 64), f32(50, 64), True, f32(40, 50), empty(sf.product_workspace(40, 50, 64), dtype=torch.uint8)], (3,)),
        "product_own": (sf.product, [f32(40, 64), f32(64, 50), False, f32(40, 50)], (3,)),
        "layernorm_param_grads": (sf.layernorm_param_grads, [x, mean, rstd, dy, new(gamma), new(gamma)], (4, 5)),
        "layer_delta_run": (sf.layer_delta_run, [numel, sf.F32, sf.F32, False, 0.0, d, plan], (5,)),
    }


NAMES = ["quant_pack", "quant_pack_fixed", "dequant_unpack", "gelu_quant_pack", "gelu_backward_dequant", "prune_scores",
         "prune_scores_threshold", "restore_scores", "softmax_prune", "softmax_backward_pruned", "prune_global_standardized",
         "prune_global_standardized_own", "layernorm_forward", "layernorm_backward", "layernorm_backward_pruned",
         "layernorm_forward_quant_pack", "layernorm_backward_dequant", "layernorm_param_grads", "layer_delta_run",
         "split_heads", "merge_heads", "product", "product_own"]


class _Subclass(torch.Tensor):
    pass


def _variants(a):
    """Other things a caller may put in an argument's place."""
    if isinstance(a, torch.Tensor):
        yield torch.nn.Parameter(a.detach(), requires_grad=False)
        yield a.as_subclass(_Subclass)
        yield a.cpu()                                                  # no GPU memory
        yield a.double() if a.is_floating_point() else a.long()        # another type
        yield a.reshape(-1)[: a.numel() // 2]                          # too small, another shape
        yield torch.stack([a, a], -1)[..., 0]                          # not contiguous
        yield a[None]                                                  # another number of dimensions
        yield None
    elif isinstance(a, bool):
        yield 1
        yield None
    elif isinstance(a, int):
        yield np.int64(a)
        yield bool(a)
        yield a + (1 << 32)                                            # wraps in 32 bits
        yield -a - 1
        yield 1 << 70
        yield float(a)
        yield None
    elif isinstance(a, float):
        yield np.float32(a)
        yield 0
        yield float("nan")
        yield "0"
    elif isinstance(a, list):
        yield tuple(a)
        yield np.array(a)
        yield []
        yield [a[0], "1"]


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("name", NAMES)
def test_both_paths_give_the_same(name, dt):
    require_gpu()
    fn, args, outs = _calls(dt)[name]
    outputs = [args[i] for i in outs]
    assert getattr(sf, "_native_" + fn.__name__)(*args, *([None] * (fn.__code__.co_argcount - len(args)))) is None     # taken
    assert _outcome(lambda: fn(*args), outputs) == _outcome(lambda: _general(fn, *args), outputs)
    names = fn.__code__.co_varnames[: len(args)]
    assert _outcome(lambda: fn(**dict(zip(names, args))), outputs) == _outcome(lambda: _general(fn, *args), outputs)
    stream = torch.cuda.current_stream().cuda_stream
    assert (_outcome(lambda: fn(*args, stream=stream), outputs) == _outcome(lambda: _general(fn, *args, stream=stream), outputs))
    for i, a in enumerate(args):
        for other in _variants(a):
            changed = list(args)
            changed[i] = other
            if isinstance(other, torch.Tensor) and other.is_cuda and i in outs:
                seen = [other if j == i else args[j] for j in outs]
            else:
                seen = outputs
            seen = [t.detach() for t in seen if t.is_contiguous() and type(t) is not _Subclass]
            got, want = _outcome(lambda: fn(*changed), seen), _outcome(lambda: _general(fn, *changed), seen)
            assert got == want, "argument %d as %r" % (i, type(other))


@pytest.mark.gpu
def test_vmap_and_current_stream():
    require_gpu()
    x = torch.randn(3, 4096, device="cuda")
    codes, scales = torch.empty(3, 2048, dtype=torch.uint8, device="cuda"), torch.empty(3, 64, device="cuda")

    def one(a):
        sf.quant_pack(a, sf.Q_BLOCK, 4, 64, 0, codes[0], scales[0])
        return a

    def outcome(f):
        try:
            torch.func.vmap(f)(x)
        except Exception as e:                                         # noqa: BLE001
            return type(e)
        return None

    assert outcome(one) is outcome(lambda a: (_general(sf.quant_pack, a, sf.Q_BLOCK, 4, 64, 0, codes[0], scales[0]), a)[1])
    # work queued on torch's current stream comes after what that stream holds already
    want, s = torch.empty_like(codes[0]), torch.cuda.Stream()
    big = torch.randn(1 << 22, device="cuda")
    sf.quant_pack(big[:4096] * 3, sf.Q_BLOCK, 4, 64, 0, want, scales[0])
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        for _ in range(20):
            big = big.clone()
        y = big[:4096] * 3
        sf.quant_pack(y, sf.Q_BLOCK, 4, 64, 0, codes[1], scales[1])
    s.synchronize()
    assert torch.equal(codes[1], want)


def test_what_is_not_on_the_gpu_is_left_to_the_general_path():
    sf.lib()
    x, codes, scales = torch.randn(256), torch.empty(128, dtype=torch.uint8), torch.empty(4)
    assert sf._native.quant_pack(x, 1, 4, 64, 0, codes, scales, None) is NotImplemented
    assert sf._native.quant_pack(x, 1, 4) is NotImplemented
    assert sf._native.layer_delta_run([1], 0, 0, False, 0.0, x, codes, None) is NotImplemented
    with pytest.raises(TypeError):
        sf._native.bind(1, 2)
