"""How the attention wrappers hand their operands to torch's batched products, on the CPU: the library's calls are
replaced by nothing, so the numbers mean nothing, and the operands are looked at instead."""
import pytest
import torch

from paper_2305_18513_amd import autograd as ag


@pytest.fixture
def products(monkeypatch):
    """The (left, right) operands of every torch.matmul that follows."""
    for name in ("quant_pack", "dequant_unpack", "softmax_prune", "restore_scores", "softmax_backward_pruned"):
        monkeypatch.setattr(ag.sf, name, lambda *args: None)
    seen, matmul = [], torch.matmul

    def spy(a, b):
        seen.append((a, b))
        return matmul(a, b)

    monkeypatch.setattr(torch, "matmul", spy)
    return seen


def _turned(*shape, dtype):
    return torch.zeros(*shape, dtype=dtype).transpose(-1, -2).contiguous().transpose(-1, -2).requires_grad_(True)


@pytest.mark.parametrize("lead", [(3,), (2, 3)])
def test_right_operands_of_bf16_products_are_laid_out(products, lead):
    dt = torch.bfloat16
    a, b = _turned(*lead, 8, 16, dtype=dt), _turned(*lead, 16, 8, dtype=dt)
    out = ag.MatmulFunction.apply(a, b)
    torch.autograd.grad(out, (a, b), _turned(*lead, 8, 8, dtype=dt).detach())
    for v_bits in (0, 8):
        s, v = _turned(*lead, 8, 16, dtype=dt), _turned(*lead, 16, 8, dtype=dt)
        out = ag.SoftmaxMatmulFunction.apply(s, v, 100000, v_bits)
        torch.autograd.grad(out, (s, v), _turned(*lead, 8, 8, dtype=dt).detach())
    assert len(products) == 9
    for _, right in products:
        assert right.is_contiguous()


def test_an_fp32_gradient_of_three_dimensions_is_multiplied_as_it_lies(products):
    s, v = torch.zeros(3, 8, 16, requires_grad=True), torch.zeros(3, 16, 8, requires_grad=True)
    grad = _turned(3, 8, 8, dtype=torch.float32).detach()
    out = ag.SoftmaxMatmulFunction.apply(s, v)
    torch.autograd.grad(out, (s, v), grad)
    (left, _), (_, right) = products[1:]
    assert left.data_ptr() == right.data_ptr() == grad.data_ptr() and not left.is_contiguous()


def test_a_gradient_of_four_dimensions_is_laid_out_once(products):
    s, v = torch.zeros(2, 3, 8, 16, requires_grad=True), torch.zeros(2, 3, 16, 8, requires_grad=True)
    grad = _turned(2, 3, 8, 8, dtype=torch.float32).detach()
    out = ag.SoftmaxMatmulFunction.apply(s, v)
    torch.autograd.grad(out, (s, v), grad)
    (left, _), (_, right) = products[1:]
    assert left.data_ptr() == right.data_ptr() != grad.data_ptr() and left.is_contiguous()
