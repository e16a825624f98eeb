"""slimfit_product and the linear layers that use it, against 64-bit products of the same operands.

Bound: fp32 additions in any order are at most K 2^-24 sum |a||b| off; the parts of an operand add up to it exactly, and what the
kernel leaves out of a product is below 2^-24 of it, whatever stands beside it in its row.  The error's 2-norm grows with the square
root of K where signs are mixed: half of sqrt(K) 2^-24 of the result's norm (an fp32 product measures 0.3 sqrt(K) 2^-24 at K = 768)."""
import numpy as np
import pytest
import torch

from paper_2305_18513_amd import autograd as ag
from paper_2305_18513_amd import binding as sf
from tests.gpu_util import require_gpu


def _operands(M, N, K, deep, seed, scale=1.0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    a = torch.randn(M, K, generator=g, device="cuda") * scale
    b = torch.randn(*((N, K) if deep else (K, N)), generator=g, device="cuda")
    return a, b


def _product(a, b, deep):
    M, N = a.shape[0], b.shape[0] if deep else b.shape[1]
    room = torch.full((M * N + 64,), 7.5, device="cuda")               # what lies behind the result stays as it is
    sf.product(a, b, deep, room[: M * N].view(M, N))
    assert bool((room[M * N:] == 7.5).all())
    return room[: M * N].view(M, N)


def _check(a, b, deep):
    bt = (b.t() if deep else b).double()
    want = a.double() @ bt
    off = (_product(a, b, deep).double() - want).abs()
    K = a.shape[1]
    assert bool((off <= (K + 1) * 2.0 ** -24 * (a.double().abs() @ bt.abs()) + 1e-300).all())
    assert float(off.norm()) <= 0.5 * K ** 0.5 * 2.0 ** -24 * float(want.norm()) + 1e-300


# tiles of 64 columns and two groups (up to 256 tiles), edges of rows, columns and depth (an odd number of steps, one step)
@pytest.mark.gpu
@pytest.mark.parametrize("deep", [True, False])
@pytest.mark.parametrize("M,N,K", [(1, 1, 32), (3, 64, 64), (127, 63, 96), (128, 65, 128), (129, 128, 160), (257, 200, 32),
                                   (640, 333, 224), (1000, 960, 256), (100, 70, 1536), (50, 90, 1568), (33, 17, 3072), (70, 40, 3136)])
def test_small(M, N, K, deep):
    require_gpu()
    _check(*_operands(M, N, K, deep, M + N + K), deep)


# 96 and 128 columns with two groups, 96 with one: sizes on either side of each change, whole tiles and ragged rows and columns
@pytest.mark.gpu
@pytest.mark.parametrize("deep", [True, False])
@pytest.mark.parametrize("M,N,K", [(4096, 512, 96), (4096, 520, 96), (4000, 768, 160), (4096, 769, 64), (4090, 1021, 96),
                                   (4096, 1025, 64), (4100, 1000, 160), (4001, 1500, 96), (2040, 3001, 32), (4000, 2200, 96), (9000, 1500, 32),
                                   (4096, 3072, 64), (4090, 3000, 96)])
def test_large(M, N, K, deep):
    require_gpu()
    _check(*_operands(M, N, K, deep, M + N + K), deep)


@pytest.mark.gpu
@pytest.mark.parametrize("deep", [True, False])
def test_rows_of_unlike_size(deep):
    """Rows and columns of any scale, and entries of a row spread over many binades or beside one that meets zeros."""
    require_gpu()
    a, b = _operands(300, 200, 256, deep, 5)
    g = torch.Generator(device="cuda").manual_seed(6)
    rows = torch.exp(torch.randn(300, 1, generator=g, device="cuda") * 10)
    a, rows = a * rows, (b if deep else b.t())
    rows *= torch.exp(torch.randn(200, 1, generator=g, device="cuda") * 8)
    want = a.double() @ rows.double().t()
    off = (_product(a, b, deep).double() - want).abs()
    assert bool((off <= 266 * 2.0 ** -24 * (a.double().abs() @ rows.double().abs().t()) + 256 * 2.0 ** -149).all())
    wide = a * torch.exp(torch.randn(300, 256, generator=g, device="cuda") * 2)
    _check(wide, b, deep)
    for large in (1e8, 1e11, 1e20):                                    # an entry that meets zeros takes no bits from its row's others
        a[:, 5], rows[:, 5] = large, 0.0
        _check(a, b, deep)


@pytest.mark.gpu
@pytest.mark.parametrize("deep", [True, False])
def test_the_whole_range_of_fp32(deep):
    """Subnormal rows against columns near the largest numbers, the reverse, and both small: no bits are lost on the way."""
    require_gpu()
    a, b = _operands(200, 100, 96, deep, 7)
    rows = b if deep else b.t()
    for up, down in ((2.0 ** -142, 2.0 ** 124), (2.0 ** -110, 2.0 ** 60), (2.0 ** -120, 1.0), (2.0 ** -60, 2.0 ** -70), (2.0 ** 110, 2.0 ** -100),
                     (2.0 ** 60, 2.0 ** 40)):
        x, y = (a.double() * up).float(), (rows.double() * down).float()
        y = y.contiguous() if deep else y.t().contiguous()
        yt = (y.t() if deep else y).double()
        off = (_product(x, y, deep).double() - x.double() @ yt).abs()
        assert bool((off <= 97 * 2.0 ** -24 * (x.double().abs() @ yt.abs()) + 2.0 ** -149).all()), (up, down)


@pytest.mark.gpu
def test_scales_and_zeros():
    require_gpu()
    for scale in (1e-12, 1e-6, 1e10, 1e25):
        _check(*_operands(200, 100, 128, True, 3, scale), True)
    a, b = _operands(200, 100, 128, True, 4)
    a[5:50] = 0.0
    out = _product(a, b, True)
    assert bool((out[5:50] == 0).all())
    # whole numbers whose sums fit 24 bits are exact
    a, b = (torch.randint(-500, 500, t.shape, device="cuda").float() for t in (a, b))
    assert torch.equal(_product(a, b, True).double(), a.double() @ b.double().t())


@pytest.mark.gpu
@pytest.mark.parametrize("deep", [True, False])
@pytest.mark.parametrize("M,N,K", [(150, 100, 96), (4100, 1000, 64)])
def test_not_finite(M, N, K, deep):
    """Rows and columns that hold infinities, NaN or the largest numbers come out as plain arithmetic has them; the others
    are not touched by them."""
    require_gpu()
    a, b = _operands(M, N, K, deep, 9)
    rows = b if deep else b.t()
    a[1, 3], a[2, 5], a[40, 7], a[M - 1, 0] = float("inf"), float("nan"), 3.4e38, -float("inf")
    rows[17, 9], rows[N - 1, K - 1] = -3.4e38, float("inf")
    rows[17, 7] = 0.25
    got, ref = _product(a, b, deep), a.cpu() @ (b.cpu().t() if deep else b.cpu())
    got = got.cpu()
    plain = torch.isfinite(ref) & (ref.abs() < 1e30)
    keep = torch.ones(M, N, dtype=torch.bool)
    keep[[1, 2, 40, M - 1]], keep[:, [17, N - 1]] = False, False
    assert bool((plain | ~keep).all()) and bool(torch.isfinite(got[keep]).all())
    # two fp32 sums of K products of entries below 6
    assert float((got[keep] - ref[keep]).abs().max()) <= 2 * (K + 1) * 2.0 ** -24 * 36 * K
    assert torch.equal(torch.isnan(got[1, :16]), torch.isnan(ref[1, :16])) and torch.equal(got[1, :16], ref[1, :16])      # inf times finite
    assert bool(torch.isnan(got[2]).all())
    assert torch.allclose(got[40, :16], ref[40, :16], rtol=1e-5)       # 3.4e38 times less than one, or an overflow
    assert torch.equal(torch.isinf(got[:, N - 1]) & keep.any(1), torch.isinf(ref[:, N - 1]) & keep.any(1))


@pytest.mark.gpu
@pytest.mark.parametrize("deep", [True, False])
@pytest.mark.parametrize("M,N,K", [(150, 100, 96), (4100, 1000, 64), (2100, 3000, 32)])
def test_nothing_finite(M, N, K, deep):
    """Whole operands of NaN, and of infinities and finite numbers in turn, come out element by element as fp32 sums do."""
    require_gpu()
    a, b = _operands(M, N, K, deep, 11)
    assert bool(torch.isnan(_product(torch.full_like(a, float("nan")), b, deep)).all())
    a[::2] = float("inf")
    got, ref = _product(a, b.abs() + 0.5, deep).cpu(), a.cpu() @ (b.cpu().t() if deep else b.cpu()).abs().add(0.5)
    assert bool((got[::2] == float("inf")).all()) and bool(torch.isfinite(got[1::2]).all())
    assert float((got[1::2] - ref[1::2]).abs().max()) <= 2 * (K + 1) * 2.0 ** -24 * 36 * K


@pytest.mark.gpu
def test_what_is_not_finite_takes_little_longer():
    """A step that has diverged (every entry NaN) takes two to three times an ordinary one's time, not the 130 of an output at a time."""
    require_gpu()
    a, b = _operands(4096, 768, 768, True, 12)
    out = torch.empty(4096, 768, device="cuda")

    def took(x):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        sf.product(x, b, True, out)
        start.record()
        for _ in range(10):
            sf.product(x, b, True, out)
        end.record()
        torch.cuda.synchronize()
        return start.elapsed_time(end)

    assert took(torch.full_like(a, float("nan"))) < 20 * took(a)


@pytest.mark.gpu
def test_refused_and_empty():
    require_gpu()
    t = lambda *s: torch.zeros(*s, device="cuda")                      # noqa: E731
    sf.product(t(0, 32), t(5, 32), True, t(0, 5))
    sf.product(t(5, 32), t(0, 32), True, t(5, 0))
    for K in (0, 31, 40):
        with pytest.raises(RuntimeError):
            sf.product(t(4, K), t(4, K), True, t(4, 4))
    for a, b, deep, out in ((t(4, 32), t(4, 64), True, t(4, 4)), (t(4, 32), t(4, 32), False, t(4, 32)), (t(4, 32), t(4, 32), True, t(4, 5)),
                            (t(4, 32).double(), t(4, 32), True, t(4, 4))):
        with pytest.raises(Exception):
            sf.product(a, b, deep, out)


# ---- the linear layer: which products are the library's, and that the others stay torch's

def _calls(monkeypatch):
    seen, real = [], sf.product
    monkeypatch.setattr(sf, "product", lambda *a: (seen.append(a[2]), real(*a))[1])
    return seen


@pytest.mark.gpu
def test_linear_layers(monkeypatch):
    require_gpu()
    seen = _calls(monkeypatch)
    g = torch.Generator(device="cuda").manual_seed(1)
    w = torch.randn(768, 512, generator=g, device="cuda")
    x = torch.randn(2, 2048, 512, generator=g, device="cuda", requires_grad=True)
    y = ag.LinearFunction.apply(x, w, None)
    dy = torch.randn(2, 2048, 768, generator=g, device="cuda")
    (dx,) = torch.autograd.grad(y, x, dy)
    assert seen == [True, False]
    for got, want in ((y, x.double() @ w.double().t()), (dx, dy.double() @ w.double())):
        assert bool((got.double() - want).norm() <= 0.5 * 768 ** 0.5 * 2.0 ** -24 * want.norm())
    # a gradient that is to be differentiated again, strides, other types, other devices, few rows, a bias
    seen.clear()
    y = ag.LinearFunction.apply(x, w, None)
    (dx,) = torch.autograd.grad(y, x, dy.requires_grad_(True), create_graph=True)
    assert dx.requires_grad and seen == [True]
    seen.clear()
    with torch.no_grad():
        for xx, ww, bias in ((x.transpose(0, 1), w, None), (x.bfloat16(), w.bfloat16(), None),
                             (x.view(1024, 2048), w.view(192, 2048), None),
                             (x, w, torch.zeros(768, device="cuda")), (x[..., :511], w[:, :511], None), (x, w.t().contiguous().t(), None),
                             (torch.randn(4096, 512), torch.randn(768, 512), None)):
            want = torch.nn.functional.linear(xx, ww, bias)
            assert torch.equal(ag.LinearFunction.apply(xx, ww, bias), want)
        with torch.autocast("cuda", dtype=torch.bfloat16):
            assert ag.LinearFunction.apply(x, w, None).dtype == torch.bfloat16
    assert seen == []


@pytest.mark.gpu
def test_captured_linear_layers_are_the_eager_ones(monkeypatch):
    """Which product a layer takes goes by its sizes alone: a captured step has the bits of an eager one, small or large."""
    require_gpu()
    seen = _calls(monkeypatch)
    g = torch.Generator(device="cuda").manual_seed(1)
    for rows, columns, library in ((70, 50, False), (200, 130, True), (1024, 768, False), (1800, 768, True)):
        x, w = (torch.randn(n, 768, generator=g, device="cuda") for n in (rows, columns))
        seen.clear()
        with torch.no_grad():
            want = ag.LinearFunction.apply(x, w, None)
            off = (want.double() - x.double() @ w.double().t()).norm() / want.double().norm()
            assert seen == [True] * library and float(off) <= 0.5 * 768 ** 0.5 * 2.0 ** -24
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                ag.LinearFunction.apply(x, w, None)                    # torch's own first call is not captured
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                y = ag.LinearFunction.apply(x, w, None)
            assert seen == [True] * 3 * library
            for _ in range(3):
                y.zero_()
                graph.replay()
                torch.cuda.synchronize()
                assert torch.equal(y, want)


@pytest.mark.gpu
def test_products_that_are_watched_are_torchs(monkeypatch):
    """Batched gradients, forward-mode tangents of a gradient, dispatch modes and negated views reach torch's product."""
    from torch.autograd import forward_ad as fw
    from torch.utils.flop_counter import FlopCounterMode
    require_gpu()
    seen = _calls(monkeypatch)
    g = torch.Generator(device="cuda").manual_seed(2)
    w = torch.randn(768, 512, generator=g, device="cuda")
    x = torch.randn(4096, 512, generator=g, device="cuda", requires_grad=True)
    dy, tangent = (torch.randn(4096, 768, generator=g, device="cuda") for _ in range(2))
    y = ag.LinearFunction.apply(x, w, None)
    assert seen == [True]
    (both,) = torch.autograd.grad(y, x, torch.stack([dy, tangent]), is_grads_batched=True, retain_graph=True)
    torch.testing.assert_close(both, torch.stack([dy @ w, tangent @ w]))
    with fw.dual_level():
        (dx,) = torch.autograd.grad(y, x, fw.make_dual(dy, tangent), retain_graph=True)
        torch.testing.assert_close(fw.unpack_dual(dx).tangent, tangent @ w)
    with FlopCounterMode(display=False) as counter:
        torch.autograd.grad(y, x, dy, retain_graph=True)
    assert counter.get_total_flops() == 2 * 4096 * 768 * 512
    (dx,) = torch.autograd.grad(y, x, torch._neg_view(dy), retain_graph=True)
    torch.testing.assert_close(dx, -(dy @ w))
    # a gradient of zeros that autograd holds without memory
    (dx,) = torch.autograd.grad(y, x, torch._efficientzerotensor(4096, 768, device="cuda"))
    assert dx.shape == x.shape and not dx.any()
    assert seen == [True]


@pytest.mark.gpu
def test_linear_layers_take_no_memory_but_their_results():
    """Forward and backward allocate the result and nothing of the operands' size beside it."""
    require_gpu()
    x = torch.randn(4096, 3072, device="cuda", requires_grad=True)
    w, dy = torch.randn(768, 3072, device="cuda"), torch.randn(4096, 768, device="cuda")

    def peak(f):
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        out = f()
        torch.cuda.synchronize()
        return out, torch.cuda.max_memory_allocated() - before

    y, forward = peak(lambda: ag.LinearFunction.apply(x, w, None))
    _, backward = peak(lambda: torch.autograd.grad(y, x, dy))
    assert forward <= 4 * 4096 * 768 + (1 << 20) and backward <= 4 * 4096 * 3072 + (1 << 20)


@pytest.mark.gpu
def test_captured_and_replayed():
    require_gpu()
    a, b = _operands(4100, 1000, 160, True, 5)
    out, want = torch.empty(4100, 1000, device="cuda"), _product(a, b, True)
    sf.product(a, b, True, out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sf.product(a, b, True, out)
    for _ in range(3):
        out.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        torch.cuda.synchronize()


# ---- without a GPU: arguments are looked at before anything is launched

def test_arguments():
    import ctypes as C
    lib = sf.lib()
    call = lambda a, b, M, N, K, out, work=16, size=1 << 40: lib.slimfit_product(              # noqa: E731
        C.c_void_p(a), C.c_void_p(b), C.c_int32(1), C.c_int64(M), C.c_int64(N), C.c_int64(K), C.c_void_p(out), C.c_void_p(work),
        C.c_size_t(size), None)
    assert call(16, 16, -1, 4, 32, 16) == call(16, 16, 4, 4, -32, 16) == sf.ERR_INVALID_ARG
    assert call(None, None, 0, 4, 32, None) == call(None, None, 4, 0, 32, None) == sf.OK
    assert call(16, 16, 4, 4, 33, 16) == call(16, 16, 4, 4, 0, 16) == sf.ERR_UNSUPPORTED
    assert call(None, 16, 4, 4, 32, 16) == call(16, None, 4, 4, 32, 16) == call(16, 16, 4, 4, 32, None) == sf.ERR_INVALID_ARG
    assert call(4, 16, 4, 4, 32, 16) == call(16, 8, 4, 4, 32, 16) == call(16, 16, 4, 4, 32, 2) == sf.ERR_ALIGNMENT
    assert sf.product_workspace(4, 4, 32) == 0
    assert call(16, 16, 1 << 40, 1 << 40, 1 << 20, 16) == call(16, 16, 1 << 30, 1 << 20, 32, 16) == sf.ERR_UNSUPPORTED


def test_a_precision_that_the_program_chose_is_torchs():
    """set_float32_matmul_precision and its kin say what becomes of these layers' products, as of any other."""
    assert torch.get_float32_matmul_precision() == "highest"
    with torch.no_grad():
        assert not ag._watched()
        try:
            for precision in ("high", "medium"):
                torch.set_float32_matmul_precision(precision)
                assert ag._watched()
        finally:
            torch.set_float32_matmul_precision("highest")
        assert not ag._watched()


def test_which_products_are_the_librarys():
    """By sizes alone: few tiles, padding, depths of weights that lie K x N, tall products of few columns, single steps of depth."""
    for M, N, K, transposed, want in ((1792, 768, 768, True, True), (1791, 768, 768, True, False),
                                      (1024, 768, 768, True, False), (1792, 768, 1536, False, True), (1792, 768, 1568, False, False),
                                      (1792, 768, 1568, True, True), (2219, 768, 3072, False, True), (260, 6144, 1024, True, False),
                                      (400, 6000, 1024, True, True), (130, 12288, 768, False, False), (4096, 768, 3072, False, True),
                                      (256, 256, 256, True, True), (257, 256, 256, True, False), (256, 256, 1024, True, False),
                                      (192, 64, 64, False, True), (191, 64, 64, False, False), (192, 64, 32, False, False),
                                      (32768, 128, 512, True, True), (32769, 128, 512, True, False), (40000, 64, 2048, False, False),
                                      (32769, 128, 480, False, True), (32769, 129, 512, True, False), (32769, 192, 512, True, True),
                                      (17000, 128, 32, True, False), (17000, 128, 64, True, True)):
        assert ag._quicker(M, N, K, transposed) == want, (M, N, K, transposed)


def test_rows_that_the_library_refuses_are_torchs(monkeypatch):
    """A linear layer's rows are as many as torch takes: past the library's limit they never reach it."""
    asked = []
    monkeypatch.setattr(sf, "product", lambda a, b, deep, out: asked.append((a.shape[0], b.shape[0 if deep else 1])))
    monkeypatch.setattr(ag, "_plain", lambda t: True)
    monkeypatch.setattr(torch.Tensor, "get_device", lambda t: 0)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    with torch.no_grad():
        for rows, columns in ((1 << 20, 64), (34_000_000, 64), (1 << 29, 64), ((1 << 29) + 1, 64), (1 << 29, 128), (1 << 33, 64)):
            x, w = torch.empty(rows, 64, device="meta"), torch.empty(columns, 64, device="meta")
            ag._dense(x, w, True)
            ag._dense(x, w.t(), False)
    assert asked == [(1 << 20, 64)] * 2 + [(34_000_000, 64)] * 2 + [(1 << 29, 64)] * 2
    for M, N in asked:
        assert sf.product_workspace(M, N, 64) == 0                     # it takes them


def test_linear_layers_on_the_cpu_are_torchs():
    x, w = torch.randn(4096, 96, requires_grad=True), torch.randn(800, 96)
    y = ag.LinearFunction.apply(x, w, None)
    (dx,) = torch.autograd.grad(y.sum(), x)
    assert torch.equal(y, torch.nn.functional.linear(x, w)) and np.allclose(dx[0].numpy(), w.sum(0).numpy(), rtol=1e-4, atol=1e-4)
