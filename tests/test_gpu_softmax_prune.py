"""GPU parity: slimfit_softmax_prune vs the CPU oracle.  The kept columns (decided on the logits) must
be identical; probabilities and kept values are fp32 evaluations compared with the fp64 oracle within
the tolerance the header states."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2305_18513_amd import binding as sf
from paper_2305_18513_amd import synth
from tests.gpu_util import Guarded, require_gpu, to_np

pytestmark = pytest.mark.gpu


def _wide(a):
    if a.dtype == np.uint16:
        return (a.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    return a.astype(np.float64)


def _run_both(l: torch.Tensor, k: int):
    rows, cols = l.shape
    bf16 = l.dtype == torch.bfloat16
    probs = Guarded(rows * cols, l.dtype)
    vals = Guarded(rows * k, l.dtype)
    idx = Guarded(rows * k, torch.uint16)
    before = l.clone()
    sf.softmax_prune(l, k, probs.t.view(rows, cols), vals.t.view(rows, k), idx.t.view(rows, k))
    torch.cuda.synchronize()
    probs.check(); vals.check(); idx.check()
    assert torch.equal(l.view(torch.uint8), before.view(torch.uint8))

    lh = to_np(l)
    # exact probabilities: ask the oracle in fp32 storage of the widened logits so that, for bf16, only the
    # kernel's own output rounding is inside the tolerance
    lw32 = _wide(lh).astype(np.float32)
    op, _, oi = ref.softmax_prune(lw32, k, threads=4)
    _, _, oi_native = ref.softmax_prune(lh, k, want_probs=False, threads=4)
    np.testing.assert_array_equal(oi, oi_native)
    gi = to_np(idx.t).reshape(rows, k)
    np.testing.assert_array_equal(gi, oi)                                       # bit-exact decision
    want = op.astype(np.float64)
    gap = _wide(lh).max(axis=1, keepdims=True) - _wide(lh)
    tol = want * (2e-6 + 2e-7 * gap) + (want * 2.0 ** -8 if bf16 else 0.0) + 1.2e-38        # subnormal results may be flushed
    gp = _wide(to_np(probs.t)).reshape(rows, cols)
    bad = np.abs(gp - want) > tol
    assert not bad.any(), "probabilities: %d outside tolerance, worst ratio %.3g" % (
        int(bad.sum()), float((np.abs(gp - want) / tol).max()))
    # kept values are the same numbers the dense row holds
    np.testing.assert_array_equal(to_np(vals.t).reshape(rows, k),
                                  np.take_along_axis(to_np(probs.t).reshape(rows, cols), gi.astype(np.int64), axis=1))
    if not bf16:
        assert np.all(np.abs(gp.sum(axis=1) - 1.0) < 2e-6)


SHAPES = [(1, 1, 1), (7, 5, 2), (7, 5, 5), (33, 64, 6), (65, 70, 69), (130, 128, 12), (257, 197, 9),
          (101, 384, 38), (40, 577, 57), (19, 1024, 102), (1001, 256, 32), (37, 208, 20), (130, 16, 3), (9, 17, 17),
          (11, 1025, 102), (9, 1536, 153), (7, 2000, 64), (5, 2048, 204), (3, 2048, 2048)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,cols,k", SHAPES)
def test_random_rows_ties_and_ranges(rows, cols, k, dtype):
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(rows * 11 + cols)
    l = torch.randn(rows, cols, generator=g, device="cuda") * 2
    if rows > 5:
        l[1] = -3.25                                                       # all equal
        l[2] = torch.randint(-2, 3, (cols,), generator=g, device="cuda").float()      # ties across the cut
        l[3] = l[3] * 10                                                   # wide range: tiny probabilities
        l[4] = l[4] + 500.0                                                # large offset, no overflow
        l[5] = -l[5].abs() - 80.0
    _run_both(l.to(dtype), k)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,cols,k", [(1, 8, 1), (15, 197, 9), (16, 197, 9), (17, 197, 9), (33, 250, 9), (64, 256, 2),
                                         (31, 100, 6), (1037, 197, 9), (129, 3, 2), (70, 65, 4)])
def test_short_rows_several_rows_a_wavefront(rows, cols, k, dtype):
    """Rows of at most 256 columns that keep few entries take the kernel that gives a wavefront 16 or 32 rows at
    once: ragged row counts, logits of either sign, ties, and fp32 logits that only their lowest bits tell apart.
    From 128 columns on it takes them only in number, so there the rows are run alone and among 60 000 (fp32) or 20 000
    (bf16; multiples of 32: the remainder is the test's own); 256 columns always take the other kernel."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(rows * 7 + cols * 3 + k)
    l = torch.randn(rows, cols, generator=g, device="cuda") * 3
    if rows > 8:
        l[1] = -l[1].abs() - 2.0                                           # every logit negative
        l[2] = torch.randint(-1, 2, (cols,), generator=g, device="cuda").float()      # ties across the cut, zeros
        l[3] = 0.0
        low = torch.randint(0, 256, (cols,), generator=g, device="cuda", dtype=torch.int32)
        l[4] = (torch.full((cols,), 0x3F800000, dtype=torch.int32, device="cuda") + low).view(torch.float32)   # 1 + j 2^-23
        l[5] = -l[4]
        l[6] = l[6] + 300.0
    _run_both(l.to(dtype), k)
    if 128 <= cols < 256:
        more = torch.randn(60000 if dtype == torch.float32 else 20000, cols, generator=g, device="cuda") * 3
        _run_both(torch.cat([l, more]).to(dtype), k)


@pytest.mark.parametrize("cols,k", [(197, 12), (128, 16), (250, 13)])
def test_short_bf16_rows_keep_up_to_sixteen(cols, k):
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(cols + k)
    l = (torch.randn(20200, cols, generator=g, device="cuda") * 0.5).to(torch.bfloat16)      # many tied logits; enough rows
    _run_both(l, k)
    _run_both(l[:200], k)


def test_argument_errors():
    require_gpu()
    l = torch.randn(8, 2049, device="cuda")
    p = torch.empty_like(l)
    v = torch.empty(8, 4, device="cuda")
    i = torch.empty(8, 4, dtype=torch.uint16, device="cuda")
    with pytest.raises(sf.SlimfitError) as e:
        sf.softmax_prune(l, 4, p, v, i)
    assert e.value.status == sf.ERR_UNSUPPORTED
    l = torch.randn(8, 64, device="cuda")
    with pytest.raises(sf.SlimfitError) as e:
        sf.softmax_prune(l, 4, l, v, i)                                    # in place
    assert e.value.status == sf.ERR_INVALID_ARG
    with pytest.raises(sf.SlimfitError) as e:
        sf.softmax_prune(l, 65, torch.empty_like(l), torch.empty(8, 65, device="cuda"),
                         torch.empty(8, 65, dtype=torch.uint16, device="cuda"))
    assert e.value.status == sf.ERR_INVALID_ARG


@pytest.mark.parametrize("ci", [1, 2, 3, 4])
def test_attention_logits_at_full_size(ci):
    """Logits whose softmax is the attention-probability tensor of the configuration (N(0,1)/sqrt(32))."""
    require_gpu()
    cfg = synth.CONFIGS[ci]
    rows = min(cfg.score_rows, 120_000)                # the oracle's row loop stays in seconds
    g = torch.Generator(device="cuda").manual_seed(100 + ci)
    l = (torch.randn(rows, cfg.score_cols, generator=g, device="cuda") / 32 ** 0.5).to(cfg.act_dtype)
    _run_both(l, cfg.keep_k)


@pytest.mark.parametrize("ci", [3, 4])
def test_fused_kept_sets_differ_from_the_two_step_form_only_on_rounding_ties(ci):
    """softmax_prune decides on the logits; softmax followed by prune_scores decides on the rounded probabilities.
    Whole score tensor of the configuration: wherever the two kept sets differ, the rounded probabilities of the
    columns they disagree on are equal (the logits differ, their probabilities round to the same value), i.e. the
    multisets of kept values coincide.  The count of such rows goes to the design notes."""
    require_gpu()
    cfg = synth.CONFIGS[ci]
    g = torch.Generator(device="cuda").manual_seed(100 + ci)
    rows, cols, k = cfg.score_rows, cfg.score_cols, cfg.keep_k
    logits = (torch.randn(rows, cols, generator=g, device="cuda") * cfg.logit_sigma).to(cfg.act_dtype)
    probs = torch.empty_like(logits)
    v1 = torch.empty(rows, k, dtype=logits.dtype, device="cuda")
    i1 = torch.empty(rows, k, dtype=torch.uint16, device="cuda")
    sf.softmax_prune(logits, k, probs, v1, i1)
    v2, i2 = torch.empty_like(v1), torch.empty_like(i1)
    sf.prune_scores(probs, k, sf.PRUNE_TOPK, 0.0, v2, i2, None)
    torch.cuda.synchronize()
    differ = (i1.view(torch.int16) != i2.view(torch.int16)).any(dim=1)
    n_differ = int(differ.sum())
    print("config %d: %d of %d rows keep different columns in the fused and the two-step form" % (ci, n_differ, rows))
    if n_differ:
        a = torch.sort(v1[differ].float(), dim=1).values
        b = torch.sort(v2[differ].float(), dim=1).values
        assert torch.equal(a, b)                                   # same kept values: only tied columns were swapped
    # fp32 probabilities of 384 random logits almost never tie; bf16 ones (about 300 distinct values a row) often do
    assert n_differ < (rows // 1000 if cfg.act_dtype == torch.float32 else rows)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,cols,k", [(8192 * 2 + 5, 72, 20), (8192 * 5 + 3, 224, 22), (8192 * 8 + 1, 65, 17),
                                         (8192 * 2 + 1, 384, 38)])
def test_rows_a_wave_takes(rows, cols, k, dtype):
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    _run_both(torch.randn(rows, cols, generator=g, device="cuda").to(dtype), k)


@pytest.mark.parametrize("dtype,cols,k,rows", [(torch.float32, 197, 9, 60000), (torch.float32, 197, 9, 59999), (torch.float32, 160, 8, 60003),
                                               (torch.float32, 64, 6, 1000), (torch.float32, 250, 5, 60001), (torch.bfloat16, 197, 16, 20001),
                                               (torch.bfloat16, 256, 12, 20000), (torch.bfloat16, 150, 3, 19999)])
def test_short_rows_by_row_count_and_stride(dtype, cols, k, rows):
    """Both sides of the row counts and strides at which short rows change kernels."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(cols + rows)
    l = torch.randn(rows, cols, generator=g, device="cuda")
    l[100:200] = (l[100:200] * 2).round() / 2                          # ties
    l[200:300] = -l[200:300].abs() - 1.0
    _run_both(l.to(dtype), k)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cols,k", [(40, 17), (64, 20), (130, 17), (384, 38), (512, 64), (700, 65), (1100, 110)])
def test_hard_rows_for_the_value_bins(cols, k, dtype):
    """Rows whose range says nothing about the cut: masked entries, one far outlier, constant rows and maxima, ranges
    of a few denormals or of the whole type, values closer together than a bin can tell."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(cols)
    l = torch.randn(260, cols, generator=g, device="cuda")
    l[0:20, cols * 7 // 10:] = -1e9
    l[20:40, k + 1:] = -3e38                                           # hardly more left than are kept
    l[40:50, 5] = 300.0
    l[50:60] = 1.25
    l[60:70] = l[60:70].clamp(max=0.5)                                 # many equal maxima
    l[70:80] = l[70:80] * 1e-41
    l[80:90] = torch.sign(l[80:90]) * 3e38
    l[90:100] = 1000.0 + l[90:100] * 1e-3
    l[100:110] = -1000.0 + (l[100:110] * 4).round() * 2.0 ** -13
    l[110:120] = (l[110:120] * 2).round() / 2
    l[120:130] = torch.where(l[120:130] > 0, 0.0, -0.0)
    l[130:140] = l[130:140].abs() + 1e-3
    l[140:150] = -l[140:150].abs()
    l[150:160] = torch.exp(l[150:160] * 8.0).clamp(max=1e30)
    _run_both(l.to(dtype), k)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cols", [17, 64, 65, 95, 96, 97, 127, 128, 129, 192, 208, 209, 224, 225, 255])
def test_short_rows_around_the_widths_that_change_kernels(cols, dtype):
    """Lanes to a row change at 96 columns, the registers that hold a lane's part at 64, 128 and 224; the last lane's
    part is shorter or missing.  A ragged number of rows; from 128 columns on as many as the kernel is for, and one row
    below that."""
    require_gpu()
    bf16 = dtype == torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(cols)
    rows = (20000 if bf16 else 24000) + 5 if cols >= 128 else 77
    for k in (1, 9, 16) if bf16 else (1, 9):
        l = torch.randn(rows, cols, generator=g, device="cuda") * 3
        l[1] = -l[1].abs() - 2.0
        l[2] = torch.randint(-1, 2, (cols,), generator=g, device="cuda").float()
        l[3], l[4] = 0.0, 2.5
        l[5, cols // 2:] = -1e9                                            # masked columns
        l[6, cols - 2:] = 40.0                                             # the largest in the last lane's part
        l[7] = (torch.full((cols,), 0x3F800000, dtype=torch.int32, device="cuda")
                + torch.arange(cols, dtype=torch.int32, device="cuda") % 7).view(torch.float32)     # 1 + j 2^-23
        _run_both(l.to(dtype), k)
        if cols in (129, 255) and k == 9:
            _run_both(l[: rows - 6].to(dtype), k)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cols", [33, 64, 95, 127, 130, 197, 208, 255])
def test_short_rows_whose_cut_is_at_or_below_zero(cols, dtype):
    """Just as many, one more and one fewer unsigned logits than are kept: which selection runs goes by their number.  Zeros of
    both signs at the cut, all rows of a wave and one of them, signed NaN-free extremes."""
    require_gpu()
    rows = 24000 + 7 if cols >= 128 else 45
    g = torch.Generator(device="cuda").manual_seed(cols)
    k = 9
    for base in (torch.randn(rows, cols, generator=g, device="cuda") * 3, -torch.rand(rows, cols, generator=g, device="cuda") - 0.5):
        l = base.clone()
        for r, n in ((1, k - 1), (2, k), (3, k + 1)):
            l[r] = -l[r].abs() - 0.25
            l[r, torch.randperm(cols, generator=g, device="cuda")[:n]] = torch.arange(1.0, n + 1, device="cuda")
        l[4], l[5] = 0.0, -0.0
        l[6, ::2] = 0.0
        l[6, 1::2] = -0.0
        l[7] = -l[7].abs() - 1.0
        l[7, cols - k:] = 0.0
        l[8] = -1e9
        l[8, :k] = -1.0
        l[9] = -3.0e38
        l[rows - 1] = -l[rows - 1].abs() - 1.0
        _run_both(l.to(dtype), k)


@pytest.mark.parametrize("cols,rows", [(12, 32769), (64, 32768), (64, 32767), (95, 32770), (96, 32771), (97, 65536), (97, 65535), (127, 65537),
                                       (128, 65536), (129, 65538), (192, 65536), (197, 65536), (224, 65539), (255, 65541), (256, 65536)])
def test_fp32_rows_that_keep_ten_to_twelve(cols, rows):
    """Longer lists, on as many rows as the short-row kernel takes them for and on one fewer."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(cols)
    for k in (10, 12):
        l = torch.randn(rows, cols, generator=g, device="cuda") * 3
        l[1] = -l[1].abs() - 2.0
        l[2] = torch.randint(-1, 2, (cols,), generator=g, device="cuda").float()
        l[3], l[4] = 0.0, 2.5
        l[5, k:] = -1e9                                                    # as many columns as are kept, the rest masked
        l[6, cols - 2:] = 40.0
        l[7] = (torch.full((cols,), 0x3F800000, dtype=torch.int32, device="cuda")
                + torch.arange(cols, dtype=torch.int32, device="cuda") % 7).view(torch.float32)     # 1 + j 2^-23
        _run_both(l, k)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cols", [12, 33, 64, 79, 96, 97, 128, 192, 197, 255])
def test_rows_of_one_value_among_others(cols, dtype):
    """One row of a wave, some and all of them constant (zeros of either sign, positive, negative); rows whose every lane
    begins with equal entries and that differ later; masked rows of fewer finite entries than are kept, whose cut is -inf."""
    require_gpu()
    rows = 65536 + 9 if cols >= 128 else 40000 + 9
    g = torch.Generator(device="cuda").manual_seed(cols)
    value = torch.tensor([0.0, -0.0, 2.5, -2.5], device="cuda")
    for k in (1, 9, 12) if dtype == torch.float32 else (9, 16):
        if k > cols:
            continue
        l = torch.randn(rows, cols, generator=g, device="cuda") * 3
        l[8:264] = value.repeat_interleave(64)[:, None]                    # whole waves
        l[264:520:16] = value.repeat(4)[:, None]                           # one row of each
        l[520:776:2] = value.repeat(32)[:, None]
        for lanes in (2, 4, 8):                                            # the first entries of every lane's part alike
            part = -(-cols // lanes)
            l[776 + lanes * 8: 784 + lanes * 8, (torch.arange(cols, device="cuda") % part) < 3] = 0.5
        l[850:860] = -1.0
        l[850:860, cols - 1] = torch.arange(-5.0, 5.0, device="cuda")      # constant but for the last
        l[860:870, max(1, k // 2):] = float("-inf")
        l[870:880] = -l[870:880].abs()
        l[870:880, : cols - max(1, k // 2)] = float("-inf")
        l[rows - 1] = 0.0
        _run_both(l.to(dtype), k)


def test_rows_of_one_value_cost_no_second_pass():
    """Zeros, a value of either sign, and zeros in one row of sixteen: a wave that meets them selects once.  (With a second
    selection and two more walks over the rows such calls took 1.5 to 2 times as long as plain ones.)"""
    require_gpu()
    rows, cols, k = 98304, 197, 9
    plain = torch.randn(rows, cols, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    some = plain.clone()
    some[::16] = 0.0
    probs = torch.empty_like(plain)
    vals, idx = torch.empty(rows, k, device="cuda"), torch.empty(rows, k, dtype=torch.uint16, device="cuda")

    def least(l):
        times = []
        for _ in range(12):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            for _ in range(10):
                sf.softmax_prune(l, k, probs, vals, idx)
            t1.record()
            torch.cuda.synchronize()
            times.append(t0.elapsed_time(t1))
        return min(times)

    least(plain)                                                           # clocks up
    base = least(plain)
    for l in (some, torch.zeros_like(plain), torch.full_like(plain, 2.5)):
        assert least(l) < 1.3 * base


@pytest.mark.parametrize("cols,line,k", [(64, 6000, 9), (96, 6000, 2), (128, 40000, 9), (192, 40000, 7), (192, 24000, 6), (128, 24000, 2),
                                         (96, 40000, 12), (100, 40000, 7), (112, 40000, 9), (113, 131072, 9), (127, 131072, 7),
                                         (97, 98304, 6), (112, 98304, 5), (96, 98304, 6)])
def test_fp32_row_counts_at_which_kernel_or_lanes_change(cols, line, k):
    """The same rows on both sides of a line: other kernel or other lanes to a row, the same result."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(cols + k)
    l = torch.randn(line, cols, generator=g, device="cuda") * 3
    l[1] = -l[1].abs() - 2.0
    l[2] = torch.randint(-1, 2, (cols,), generator=g, device="cuda").float()
    l[3], l[4] = 0.0, -2.5
    l[5, k:] = -1e9
    l[6] = (torch.full((cols,), 0x3F800000, dtype=torch.int32, device="cuda")
            + torch.arange(cols, dtype=torch.int32, device="cuda") % 7).view(torch.float32)         # 1 + j 2^-23
    _run_both(l, k)
    _run_both(l[: line - 1], k)
