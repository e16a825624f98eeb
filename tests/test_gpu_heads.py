"""GPU parity: slimfit_split_heads / slimfit_merge_heads against the reshapes and transposes they stand for.  Copies are
exact; the scaled part is one product rounded to the type."""
import numpy as np
import pytest
import torch

from paper_2305_18513_amd import autograd as ag
from paper_2305_18513_amd import binding as sf
from tests.gpu_util import Guarded, require_gpu, to_np

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1, 8), (2, 5, 3, 8), (1, 63, 2, 64), (1, 64, 1, 64), (3, 65, 2, 64), (2, 128, 4, 64), (1, 197, 3, 64), (2, 33, 1, 72),
          (1, 200, 2, 128), (5, 4, 2, 16), (1, 68, 1, 136)]


def _apart(qkv, heads, scale):
    B, T, H3 = qkv.shape
    q, k, v = (t.reshape(B, T, heads, -1).transpose(1, 2) for t in qkv.chunk(3, -1))
    return (q.float() * scale).to(qkv.dtype).contiguous(), k.transpose(-1, -2).contiguous(), v.contiguous()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,T,h,D", SHAPES)
@pytest.mark.parametrize("scale", [0.125, 0.3])
def test_split_and_merge(B, T, h, D, scale, dtype):
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(T * 7 + D)
    qkv = torch.randn(B, T, 3 * h * D, generator=g, device="cuda").to(dtype)
    qkv.view(-1)[0], qkv.view(-1)[-1] = -0.0, 1e-40
    n = B * T * h * D
    q, kt, v = Guarded(n, dtype), Guarded(n, dtype), Guarded(n, dtype)
    sf.split_heads(qkv, scale, q.t.view(B, h, T, D), kt.t.view(B, h, D, T), v.t.view(B, h, T, D))
    back = Guarded(3 * n, dtype)
    sf.merge_heads(q.t.view(B, h, T, D), kt.t.view(B, h, D, T), v.t.view(B, h, T, D), 1.0, back.t.view(B, T, 3 * h * D))
    torch.cuda.synchronize()
    for b in (q, kt, v, back):
        b.check()
    for got, want in zip((q, kt, v), _apart(qkv, h, scale)):
        np.testing.assert_array_equal(to_np(got.t).view(np.uint16), to_np(want.reshape(-1)).view(np.uint16))
    want = qkv.clone()
    want[..., : h * D] = (want[..., : h * D].float() * scale).to(dtype)
    np.testing.assert_array_equal(to_np(back.t).view(np.uint16), to_np(want.reshape(-1)).view(np.uint16))
    sf.merge_heads(q.t.view(B, h, T, D), kt.t.view(B, h, D, T), v.t.view(B, h, T, D), scale, back.t.view(B, T, 3 * h * D))
    want[..., : h * D] = (want[..., : h * D].float() * scale).to(dtype)
    assert torch.equal(back.t.view(B, T, -1), want)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,T,h", [(2, 70, 2), (1, 128, 4)])
def test_gradients_are_those_of_the_reshapes(B, T, h, dtype):
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn(B, T, 3 * h * 64, generator=g, device="cuda").to(dtype).requires_grad_(True)
    outs = ag.SplitHeadsFunction.apply(x, h, 0.125)
    ref = _apart(x, h, 0.125)
    grads = [torch.randn(o.shape, generator=g, device="cuda").to(dtype) for o in outs]
    assert all(torch.equal(a, b) for a, b in zip(outs, ref))
    (got,) = torch.autograd.grad(outs, x, [t.transpose(2, 3).contiguous().transpose(2, 3) for t in grads])      # not contiguous
    (want,) = torch.autograd.grad(ref, x, grads)
    assert torch.equal(got, want)


def test_arguments():
    require_gpu()
    qkv = torch.randn(2, 8, 3 * 2 * 6, device="cuda")
    q = torch.empty(2, 2, 8, 6, device="cuda")
    with pytest.raises(sf.SlimfitError) as e:
        sf.split_heads(qkv, 1.0, q, torch.empty(2, 2, 6, 8, device="cuda"), torch.empty_like(q))
    assert e.value.status == sf.ERR_UNSUPPORTED
    qkv, q = torch.randn(2, 8, 48, device="cuda"), torch.empty(2, 2, 8, 8, device="cuda")
    for bad in ((qkv, torch.empty(2, 2, 8, 4, device="cuda")), (qkv.bfloat16(), torch.empty(2, 2, 8, 8, device="cuda")),
                (qkv[:, :4], torch.empty(2, 2, 8, 8, device="cuda")), (qkv, torch.empty(2, 8, 2, 8, device="cuda"))):
        with pytest.raises(ValueError):
            sf.split_heads(bad[0], 1.0, q, bad[1], torch.empty_like(q))
        with pytest.raises(ValueError):
            sf.merge_heads(q, bad[1], torch.empty_like(q), 1.0, bad[0])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("hidden,heads", [(128, 2), (128, 8), (128, 4), (96, 2), (240, 3), (128, 1), (40, 5)])
def test_encoder_block_is_what_it_was_with_reshapes(monkeypatch, hidden, heads, dtype):
    """Head sizes of 64 and 16 (the factor, a power of two, goes onto q), 32, 48, 80, 128 and 8 (the products are divided): with the
    fused reordering and without it the products see the same operands."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(heads)
    params = ag.encoder_block_params(hidden, "cuda", 3, dtype)
    x = torch.randn(2, 48, hidden, generator=g, device="cuda").to(dtype).requires_grad_(True)
    dout = torch.randn(2, 48, hidden, generator=g, device="cuda").to(dtype)
    calls = []
    for name in ("split_heads", "merge_heads"):
        kept = getattr(sf, name)
        monkeypatch.setattr(ag.sf, name, lambda *args, name=name, kept=kept: (calls.append(name), kept(*args))[1])

    def run():
        out = ag.frozen_encoder_block(x, params, heads, True)
        return out, torch.autograd.grad(out, x, dout)[0]

    out, dx = run()
    assert calls == ["split_heads", "merge_heads"]
    monkeypatch.setattr(ag, "_rows_of_vectors", lambda dim, t: False)
    want, want_dx = run()
    assert len(calls) == 2                                             # the reshapes alone
    assert torch.equal(out, want) and torch.equal(dx, want_dx)


def test_heads_that_are_no_whole_vectors_keep_the_reshapes():
    require_gpu()
    params = ag.encoder_block_params(24, "cuda", 3, torch.bfloat16)
    x = torch.randn(1, 16, 24, device="cuda").bfloat16()
    assert torch.isfinite(ag.frozen_encoder_block(x, params, 2, True).float()).all()                 # 12 elements: 24 bytes
