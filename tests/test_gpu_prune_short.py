"""GPU parity of slimfit_prune_scores on short rows that keep few entries (the kernel with several rows per
wavefront): every route of it -- keys that carry the column, the exact route for rows whose cut cannot be
told from 24 value bits, signed keys -- against the CPU oracle, bit for bit.  fp32 rows of 128 columns and more take
that kernel from 20 000 rows on (and at no stride of a multiple of 64 columns), so there the rows that a test is about
stand among enough plain ones."""
import numpy as np
import pytest
import torch

from paper_2305_18513_amd import binding as sf
from tests.gpu_util import require_gpu
from tests.test_gpu_prune import _run_both

pytestmark = pytest.mark.gpu

ENOUGH = 20000             # a multiple of the rows a wave takes: the remainder is the test's own


def _among_many(p, g):
    if p.dtype != torch.float32 or p.shape[1] < 128:
        return p
    return torch.cat([p, torch.softmax(torch.randn(ENOUGH, p.shape[1], generator=g, device="cuda") * 0.5, dim=-1)])


ROWS = [1, 15, 16, 17, 31, 32, 33, 64, 1000, 1037]
COLS_K = [(1, 1), (2, 1), (3, 3), (5, 2), (16, 4), (17, 9), (63, 6), (64, 6), (65, 7), (100, 9), (128, 9),
          (197, 9), (197, 1), (199, 5), (250, 8), (255, 9), (256, 9), (256, 2)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cols,k", COLS_K)
def test_shapes_and_ragged_row_counts(cols, k, dtype):
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(cols * 131 + k)
    for rows in ROWS:
        p = torch.softmax(torch.randn(rows, cols, generator=g, device="cuda") * 0.5, dim=-1).to(dtype)
        _run_both(p, k, restore=False)
        _run_both(p, k, mode=sf.PRUNE_THRESHOLD, tau=1.3 / cols, restore=False)
        if rows in (1, 17, 1037) and dtype == torch.float32 and cols >= 128:
            many = _among_many(p, g)
            _run_both(many, k, restore=False)
            _run_both(many, k, mode=sf.PRUNE_THRESHOLD, tau=1.3 / cols, restore=False)


@pytest.mark.parametrize("cols,k", [(197, 9), (128, 12), (250, 16), (64, 13), (33, 16)])
def test_bf16_keeps_up_to_sixteen(cols, k):
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(cols + k)
    p = torch.softmax(torch.randn(333, cols, generator=g, device="cuda") * 0.3, dim=-1).to(torch.bfloat16)   # many ties
    _run_both(p, k)
    _run_both(p, k, mode=sf.PRUNE_THRESHOLD, tau=1.0 / cols)


@pytest.mark.parametrize("k", [1, 4, 9])
def test_fp32_cut_inside_one_bucket_of_24_bits(k):
    """Entries that agree in their upper 24 bits and differ below: only the full 32-bit images order them."""
    require_gpu()
    cols, rows = 197, 70
    g = torch.Generator(device="cuda").manual_seed(k)
    low = torch.randint(0, 256, (rows, cols), generator=g, device="cuda", dtype=torch.int32)
    base = torch.full((rows, cols), 0x3C000000, dtype=torch.int32, device="cuda")       # 2^-7 and the 255 floats above it
    p = (base + low).view(torch.float32).clone()
    p[10:20, ::3] *= 0.5                                            # some entries far below the bucket
    p[20:30, 5] = 1.0                                               # one far above
    p[30:40] = p[30:40, :1]                                         # constant rows
    p[40:50, 100:] = p[40:50, 99:100]                               # long runs of equal entries across lanes
    tau = float(torch.tensor(0x3C000080, dtype=torch.int32).view(torch.float32))        # a threshold inside the bucket
    for q, t in ((p, tau), (_among_many(p, g), tau), (-p, -tau), (_among_many(-p, g), -tau)):      # and among negative entries
        _run_both(q, k)
        _run_both(q, k, mode=sf.PRUNE_THRESHOLD, tau=t)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cols,k", [(197, 9), (64, 6), (130, 3)])
def test_signs_zeros_and_ties(cols, k, dtype):
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(cols + 7 * k)
    p = torch.randn(200, cols, generator=g, device="cuda")
    p[0:20] = -p[0:20].abs()                                        # all negative
    p[20:40] = (p[20:40] * 2).round() / 2                           # few distinct values, both signs
    p[40:50] = 0.0
    p[40:50, ::2] = -0.0                                            # +0 and -0 tie; the kept bits must be the entry's own
    p[50:60] = -0.0
    p[60:70, : cols // 2] = 0.0                                     # zeros at the cut below a few positive entries
    p[60:70, 0] = 1.0
    p[70:80] = p[70:80].abs() * 1e-41                               # denormals (fp32); flushed to zero patterns in bf16
    p[80:90] = -1.5
    p[90:100, 3] = float("inf")
    p[100:110, 4] = float("-inf")
    p = p.to(dtype)
    for q in (p, _among_many(p, g)) if dtype == torch.float32 and cols >= 128 else (p,):
        _run_both(q, k)
        for tau in (0.0, -0.0, -0.75, 0.5):
            _run_both(q, k, mode=sf.PRUNE_THRESHOLD, tau=tau)


def test_misaligned_rows_take_the_other_kernel_and_agree():
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(5)
    rows = ENOUGH + 77
    base = torch.softmax(torch.randn(rows, 197, generator=g, device="cuda"), dim=-1)
    flat = torch.empty(rows * 197 + 1, device="cuda")
    flat[1:] = base.reshape(-1)
    p = flat[1:].view(rows, 197)
    assert p.data_ptr() % 16 != 0
    vals = torch.empty(rows, 9, device="cuda")
    idx = torch.empty(rows, 9, dtype=torch.uint16, device="cuda")
    vals2, idx2 = torch.empty_like(vals), torch.empty_like(idx)
    sf.prune_scores(p, 9, sf.PRUNE_TOPK, 0.0, vals, idx, None)
    sf.prune_scores(base, 9, sf.PRUNE_TOPK, 0.0, vals2, idx2, None)
    torch.cuda.synchronize()
    assert torch.equal(vals, vals2) and torch.equal(idx.view(torch.int16), idx2.view(torch.int16))


@pytest.mark.parametrize("dtype,cols,k,rows", [
    (torch.float32, 197, 9, 20000), (torch.float32, 197, 9, 19999), (torch.float32, 130, 3, 20011), (torch.float32, 250, 8, 20001),
    (torch.float32, 160, 9, 20007), (torch.float32, 192, 9, 20000), (torch.bfloat16, 197, 16, 20001), (torch.bfloat16, 33, 16, 19999)])
def test_rows_enough_for_several_a_wave(dtype, cols, k, rows):
    """Both sides of the row counts and strides at which the kernel changes; fp32 rows of every hard kind among many."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(cols * 7 + k)
    p = torch.softmax(torch.randn(rows, cols, generator=g, device="cuda") * 0.5, dim=-1)
    low = torch.randint(0, 256, (600, cols), generator=g, device="cuda", dtype=torch.int32)
    p[1000:1600] = (0x3C000000 + low).view(torch.float32)            # entries that agree in their upper 24 bits
    p[1100:1200] = -p[1100:1200]
    p[1200:1300] = p[1200:1300, :1]
    p[1300:1400] = (torch.randn(100, cols, generator=g, device="cuda") * 2).round() / 2
    p[1400:1450] = 0.0
    p[1400:1450, ::2] = -0.0
    p[1450:1500] = p[1450:1500].abs() * 1e-41
    p = p.to(dtype)
    _run_both(p, k, restore=False)
    for tau in (1.3 / cols, 0.0, float(torch.tensor(0x3C000080, dtype=torch.int32).view(torch.float32))):
        _run_both(p, k, mode=sf.PRUNE_THRESHOLD, tau=tau, restore=False)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cols", [129, 130, 131, 160, 161, 197, 199, 207, 208, 209, 250, 255])
def test_rows_whose_neighbours_are_selected_together(cols, dtype):
    """bf16 rows of more than 128 columns: the walk takes entries in twos; fp32 rows one by one.  Odd and even parts, the largest entries side by side, apart,
    at the ends of the lanes' parts, equal to one another, all of them of one sign or the other."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(cols)
    bf16 = dtype == torch.bfloat16
    for k in (1, 2, 9, 16) if bf16 else (1, 2, 9):
        x = torch.softmax(torch.randn(20000 + 5, cols, generator=g, device="cuda") * 3, -1)
        lane = -(-cols // (2 if bf16 else 4))                              # entries of a lane
        ends = [c for q in range(4) for c in (q * lane - 2, q * lane - 1, q * lane, q * lane + 1) if 0 <= c < cols] + [cols - 2, cols - 1]
        x[1] = torch.arange(cols, device="cuda") / 1024.0                  # ascending: every pair's larger entry is its second
        x[2] = x[1].flip(0)
        x[3, :k] = 2.0 + torch.arange(k, device="cuda") / 64.0             # side by side
        x[4, cols - k:] = 2.0
        x[5, ::2] = 1.0                                                    # the first of every pair
        x[6, 1::2] = 1.0
        x[7, ends] = 3.0
        x[8] = -x[8] - 1.0                                                 # no positive entry
        x[9, k:] = -1.0                                                    # just as many positive ones as are kept
        x[10], x[11], x[12] = 0.5, 0.0, -0.0
        x[13, 1::2] = 0.0                                                  # masked neighbours
        _run_both(x.to(dtype), k, sf.PRUNE_TOPK, 0.0)
        _run_both(x.to(dtype), k, sf.PRUNE_THRESHOLD, 0.25)


@pytest.mark.parametrize("cols,rows", [(12, 32769), (33, 32771), (64, 32768), (64, 32767), (95, 32770), (96, 32768), (97, 65536), (97, 65535),
                                       (112, 65537), (127, 65539), (128, 65536)])
def test_fp32_rows_that_keep_ten_to_twelve(cols, rows):
    """Longer lists, on as many rows as the kernel takes them for and on one fewer; 24-bit buckets across the cut."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(cols)
    for k in (10, 12):
        x = torch.softmax(torch.randn(rows, cols, generator=g, device="cuda") * 3, -1)
        x[1] = torch.arange(cols, device="cuda") / 1024.0
        x[2] = x[1].flip(0)
        x[3], x[4] = 0.5, -0.0
        x[5] = -x[5] - 1.0
        x[6, min(k, cols - 1):] = 0.0                                      # masked from there on
        x[7, k - 1:] = -1.0
        x[8] = (torch.full((cols,), 0x3F800000, dtype=torch.int32, device="cuda")
                + torch.arange(cols, dtype=torch.int32, device="cuda") % 7).view(torch.float32)     # 1 + j 2^-23
        x[rows - 1, cols - k:] = 2.0                                       # the last row, of a wave that is not full
        _run_both(x, k, sf.PRUNE_TOPK, 0.0, restore=False)
        _run_both(x, k, sf.PRUNE_THRESHOLD, 0.25, restore=False)
