"""GPU: the largest shapes the entry points accept in practice -- tensors whose element or byte offsets
pass 2^31 and 2^32.  The oracle checks sampled units that it can compute one by one (quantisation
blocks, score rows) or closed forms; the whole-tensor pruner is checked through the properties that
define its result at any size."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2305_18513_amd import binding as sf
from tests.gpu_util import require_gpu, to_np

pytestmark = pytest.mark.gpu


def _need(gib):
    require_gpu()
    free, _ = torch.cuda.mem_get_info()
    if free < gib * (1 << 30):
        pytest.skip("needs %d GiB of free device memory" % gib)


def test_quant_dequant_past_two_to_the_32_elements():
    _need(30)
    n = (1 << 32) + 4099                                        # ragged tail, offsets beyond 32 bits
    bits, block = 4, 32
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    step = 1 << 28
    for s in range(0, n, step):                                 # generated in slices to bound temporaries
        m = min(step, n - s)
        x[s:s + m] = torch.randn(m, generator=g, device="cuda").to(torch.bfloat16)
    codes = torch.empty(sf.packed_bytes(n, bits), dtype=torch.uint8, device="cuda")
    scales = torch.empty(sf.num_blocks(n, block), dtype=torch.float32, device="cuda")
    y = torch.empty_like(x)
    sf.quant_pack(x, sf.Q_BLOCK, bits, block, 0, codes, scales)
    sf.dequant_unpack(codes, scales, sf.Q_BLOCK, bits, block, 0, y)
    torch.cuda.synchronize()
    nb = sf.num_blocks(n, block)
    rng = np.random.default_rng(0)
    picks = sorted(set([0, 1, nb - 1, nb - 2, (1 << 31) // block, (1 << 32) // block - 1, (1 << 32) // block,
                        (1 << 32) // block + 1] + rng.integers(0, nb, 300).tolist()))
    for b in picks:
        lo, hi = b * block, min((b + 1) * block, n)
        xb = to_np(x[lo:hi])
        oc, osc = ref.quant_pack(xb, mode=ref.Q_BLOCK, bits=bits, block=block)
        got_c = to_np(codes[lo * bits // 8:(hi * bits + 7) // 8])
        assert np.array_equal(got_c, oc), "codes of block %d" % b
        assert to_np(scales[b:b + 1]).view(np.uint32)[0] == osc.view(np.uint32)[0], "scale of block %d" % b
        oy = ref.dequant_unpack(oc, osc, hi - lo, mode=ref.Q_BLOCK, bits=bits, block=block, out_dtype=np.uint16)
        assert np.array_equal(to_np(y[lo:hi]), oy), "dequantised block %d" % b


def test_prune_and_restore_rows_past_two_to_the_32_elements():
    _need(60)
    rows, cols, k = 11_200_000, 384, 38                         # 4.3e9 elements, 17 GB
    g = torch.Generator(device="cuda").manual_seed(2)
    p = torch.empty(rows, cols, device="cuda")
    step = 1_400_000
    for s in range(0, rows, step):
        p[s:s + step] = torch.softmax(torch.randn(min(step, rows - s), cols, generator=g, device="cuda") / 32 ** 0.5, dim=1)
    vals = torch.empty(rows, k, device="cuda")
    idx = torch.empty(rows, k, dtype=torch.uint16, device="cuda")
    counts = torch.empty(rows, dtype=torch.int32, device="cuda")
    sf.prune_scores(p, k, sf.PRUNE_TOPK, 0.0, vals, idx, counts)
    out = torch.empty_like(p)
    sf.restore_scores(vals, idx, counts, out)
    torch.cuda.synchronize()
    assert bool((counts == k).all())
    rng = np.random.default_rng(1)
    first_past = (1 << 32) // cols
    picks = sorted(set([0, rows - 1, first_past - 1, first_past, first_past + 1, (1 << 31) // cols]
                       + rng.integers(0, rows, 400).tolist()))
    sel = torch.tensor(picks, device="cuda")
    ov, oi, _ = ref.prune_scores(to_np(p[sel]), k)
    assert np.array_equal(to_np(idx.view(torch.int16)[sel]).view(np.uint16), oi)
    assert np.array_equal(to_np(vals[sel]).view(np.uint32), ov.view(np.uint32))
    assert np.array_equal(to_np(out[sel]), ref.restore_scores(ov, oi, None, cols))
    # every row of the restored tensor holds exactly k entries, each a copy of the input's
    nz = out != 0
    assert bool((nz.sum(1) == k).all()) and bool(((out == p) | ~nz).all())


def test_softmax_backward_rows_past_two_to_the_32_elements():
    """Both kernels of slimfit_softmax_backward_pruned (a wave per row at k = 38, spread records at k = 9) on a gradient
    tensor of more than 2^32 bf16 elements: sampled rows against the oracle, and the zero pattern everywhere."""
    _need(40)
    g = torch.Generator(device="cuda").manual_seed(3)
    for cols, k in ((384, 38), (197, 9)):
        rows = ((1 << 32) + (1 << 22)) // cols
        dp = torch.empty(rows, cols, dtype=torch.bfloat16, device="cuda")
        step = 1_000_000
        for s in range(0, rows, step):
            dp[s:s + step] = torch.randn(min(step, rows - s), cols, generator=g, device="cuda").bfloat16()
        # pairs: k distinct columns per row in ascending order, values in (0, 1)
        cols_sorted = torch.empty(rows, k, dtype=torch.int16, device="cuda")
        for s in range(0, rows, step):
            m = min(step, rows - s)
            perm = torch.rand(m, cols, generator=g, device="cuda").argsort(dim=1)[:, :k]
            cols_sorted[s:s + m] = perm.sort(dim=1).values.to(torch.int16)
        idx = cols_sorted.view(torch.uint16)
        vals = torch.rand(rows, k, generator=g, device="cuda").bfloat16()
        ds = torch.empty_like(dp)
        sf.softmax_backward_pruned(vals, idx, None, dp, ds)
        torch.cuda.synchronize()
        first_past = (1 << 32) // cols
        rng = np.random.default_rng(cols)
        picks = sorted(set([0, rows - 1, first_past - 1, first_past, first_past + 1, (1 << 31) // cols]
                           + rng.integers(0, rows, 300).tolist()))
        sel = torch.tensor(picks, device="cuda")
        v32 = vals[sel].float().cpu().numpy()
        d32 = dp[sel].float().cpu().numpy()
        ih = to_np(idx.view(torch.int16)[sel]).view(np.uint16)
        want = ref.softmax_backward_pruned(v32, ih, None, d32).astype(np.float64)
        got = ds[sel].float().cpu().numpy().astype(np.float64)
        absdot = np.abs(np.take_along_axis(d32, ih.astype(np.int64), 1).astype(np.float64) * v32).sum(1, keepdims=True)
        tol = 2e-6 * absdot + np.abs(want) * 2.0 ** -8 + 1e-30
        assert np.all(np.abs(got - want) <= tol)
        # every row holds at most k non-zero entries (a product may round to zero), all at kept columns
        nz = ds != 0
        assert bool((nz.sum(1) <= k).all())
        kept = torch.zeros(len(picks), cols, dtype=torch.bool, device="cuda")
        kept.scatter_(1, cols_sorted[sel].long(), True)
        assert bool((~nz[sel] | kept).all())
        del dp, ds, nz, vals, idx, cols_sorted


def test_layer_delta_closed_form_past_two_to_the_32_elements():
    _need(40)
    n = (1 << 32) + 16384 * 3 + 5
    g = torch.Generator(device="cuda").manual_seed(3)
    w = torch.empty(n, device="cuda")
    step = 1 << 28
    for s in range(0, n, step):
        m = min(step, n - s)
        t = (torch.randn(m, generator=g, device="cuda") * 0.02).to(torch.bfloat16).float()      # 8-bit mantissas
        w[s:s + m] = torch.where(t == 0, torch.full_like(t, 0.5), t)
    cur = w * (1 + 2.0 ** -7)                                   # exact in fp32: every term is 2^-7
    small = torch.ones(1000, device="cuda")
    prev_l, cur_l = [small, w, small], [small * 1.5, cur, small.clone()]
    numel = [t.numel() for t in prev_l]
    ws = torch.empty(sf.layer_delta_workspace(numel), dtype=torch.uint8, device="cuda")
    d = torch.empty(3, device="cuda")
    sf.layer_delta(prev_l, cur_l, False, 0.0, d, ws)
    torch.cuda.synchronize()
    assert d.tolist() == [0.5, 2.0 ** -7, 0.0]


def test_whole_tensor_pruning_at_the_int32_limit():
    _need(60)
    n = (1 << 31) - 8
    k = n // 10
    g = torch.Generator(device="cuda").manual_seed(4)
    x = torch.empty(n, device="cuda")
    step = 1 << 28
    for s in range(0, n, step):
        m = min(step, n - s)
        x[s:s + m] = (torch.randn(m, generator=g, device="cuda") * 64).round() / 64      # ties at the cut are certain
    vals = torch.empty(k, device="cuda")
    idx = torch.empty(k, dtype=torch.int32, device="cuda")
    ptr = torch.empty(sf.global_tile_ptr_len(n), dtype=torch.int32, device="cuda")
    sf.prune_global(x, k, vals, idx, True, ptr)
    torch.cuda.synchronize()
    il = idx.long()
    assert int(il.min()) >= 0 and int(il.max()) < n and bool((il[1:] > il[:-1]).all())          # ascending, in range
    assert bool((x[il] == vals).all())                                                         # bit copies (no NaN here)
    T = float(vals.abs().min())
    ax = x.abs()
    above, at = int((ax > T).sum()), int((ax == T).sum())
    assert above < k <= above + at                                  # T is the k-th largest magnitude
    assert int((vals.abs() > T).sum()) == above                     # everything above it is kept
    kept_eq = il[vals.abs() == T]
    all_eq = torch.nonzero(ax == T).view(-1)
    assert torch.equal(kept_eq, all_eq[: kept_eq.numel()])          # ties go to the lowest indices
    del ax, all_eq, kept_eq
    edges = torch.arange(ptr.numel(), device="cuda", dtype=torch.int64) * sf.GLOBAL_TILE
    assert torch.equal(ptr.long(), torch.searchsorted(il, edges))
    out = torch.empty_like(x)
    sf.restore_global(vals, idx, k, out, ptr)
    torch.cuda.synchronize()
    assert int((out != 0).sum()) == int((vals != 0).sum()) and bool((out[il] == vals).all())


# A grid's threads are counted in 32 bits, and a launch of more starts fewer without an error: calls of that size go out in
# pieces.  Each is compared, around the pieces' ends and at its own, with the same call on that part alone.

def _poisoned(shape, dtype, at):
    t = torch.empty(shape, dtype=dtype, device="cuda")
    for a, b in at:
        t[a:b].view(torch.uint8).fill_(0x5A)
    return t


def test_quantiser_of_more_elements_than_a_grid_has_threads_for():
    torch.cuda.empty_cache()
    _need(160)
    n, bits, block = (1 << 35) + 5000, 4, 256
    at = [(0, 8192), ((1 << 34) - 4096, (1 << 34) + 4096), ((1 << 35) - 4096, n)]
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.empty(n, device="cuda")
    for a, b in at:
        x[a:b] = torch.randn(b - a, generator=g, device="cuda")
    kept = [x[a:b].clone() for a, b in at]
    codes = _poisoned(sf.packed_bytes(n, bits), torch.uint8, [(a // 2, b // 2) for a, b in at])
    scales = _poisoned(sf.num_blocks(n, block), torch.float32, [(a // block, -(-b // block)) for a, b in at])
    sf.quant_pack(x, sf.Q_BLOCK, bits, block, 0, codes, scales)
    torch.cuda.synchronize()
    del x
    torch.cuda.empty_cache()
    y = _poisoned(n, torch.float32, at)
    sf.dequant_unpack(codes, scales, sf.Q_BLOCK, bits, block, 0, y)
    torch.cuda.synchronize()
    for (a, b), part in zip(at, kept):
        c, s = torch.empty(sf.packed_bytes(b - a, bits), dtype=torch.uint8, device="cuda"), torch.empty(sf.num_blocks(b - a, block), device="cuda")
        sf.quant_pack(part, sf.Q_BLOCK, bits, block, 0, c, s)
        assert torch.equal(codes[a // 2: a // 2 + c.numel()], c) and torch.equal(scales[a // block: a // block + s.numel()], s)
        back = torch.empty_like(part)
        sf.dequant_unpack(c, s, sf.Q_BLOCK, bits, block, 0, back)
        assert torch.equal(y[a:b], back)
    del y, codes, scales
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_heads_of_more_sequences_than_a_grid_has_threads_for(dtype):
    torch.cuda.empty_cache()
    _need(16)
    batch, tokens, heads, dim = (1 << 21) + 3, 1, 3, 8                     # 3 * batch * heads blocks of 256 threads
    qkv = torch.randint(-99, 99, (batch, tokens, 3 * heads * dim), device="cuda", dtype=torch.int8).to(dtype)
    q, kt = torch.zeros(batch, heads, tokens, dim, dtype=dtype, device="cuda"), torch.zeros(batch, heads, dim, tokens, dtype=dtype, device="cuda")
    v = torch.zeros_like(q)
    sf.split_heads(qkv, 0.5, q, kt, v)
    parts = qkv.view(batch, tokens, 3, heads, dim)
    assert torch.equal(q, parts[:, :, 0].transpose(1, 2) * 0.5)
    assert torch.equal(kt, parts[:, :, 1].permute(0, 2, 3, 1)) and torch.equal(v, parts[:, :, 2].transpose(1, 2))
    back = torch.zeros_like(qkv)
    sf.merge_heads(q, kt, v, 2.0, back)
    assert torch.equal(back, qkv)


def test_short_rows_of_more_rows_than_a_grid_has_threads_for():
    torch.cuda.empty_cache()
    _need(80)
    rows, cols, k = (1 << 30) + 100, 2, 1
    p = torch.empty(rows, cols, device="cuda")
    p[:, 0], p[:, 1] = 0.25, 0.75
    p[5::7, 0] = 0.875
    for softmax in (False, True):
        vals, idx = torch.zeros(rows, k, device="cuda"), torch.full((rows, k), 9, dtype=torch.int16, device="cuda").view(torch.uint16)
        if softmax:
            probs = torch.zeros_like(p)
            sf.softmax_prune(p, k, probs, vals, idx)
            assert bool((probs.sum(1) - 1).abs().max() < 1e-6)
            del probs
        else:
            sf.prune_scores(p, k, sf.PRUNE_TOPK, 0.0, vals, idx, None)
            assert torch.equal(vals[:, 0], p.amax(1))
        assert torch.equal(idx.view(torch.int16)[:, 0], (p[:, 1] > p[:, 0]).to(torch.int16))
        del vals, idx
    del p
    torch.cuda.empty_cache()


def test_rows_of_a_wave_each_that_fill_a_grid_to_the_last_bit():
    """2^26 waves are 2^32 threads: a grid whose low 32 bits are zero."""
    torch.cuda.empty_cache()
    _need(190)
    rows, cols, k = 1 << 26, 320, 16
    at = [(0, 64), ((1 << 25) - 64, (1 << 25) + 64), (rows - 64, rows)]
    g = torch.Generator(device="cuda").manual_seed(6)
    l = torch.empty(rows, cols, device="cuda")
    for a, b in at:
        l[a:b] = torch.randn(b - a, cols, generator=g, device="cuda")
    probs, vals = _poisoned((rows, cols), torch.float32, at), _poisoned((rows, k), torch.float32, at)
    idx = _poisoned((rows, k), torch.uint16, at)
    sf.softmax_prune(l, k, probs, vals, idx)
    torch.cuda.synchronize()
    for a, b in at:
        part = l[a:b].clone()
        pr, v, i = torch.empty_like(part), torch.empty(b - a, k, device="cuda"), torch.empty(b - a, k, dtype=torch.uint16, device="cuda")
        sf.softmax_prune(part, k, pr, v, i)
        assert torch.equal(probs[a:b], pr) and torch.equal(vals[a:b], v) and torch.equal(idx[a:b].view(torch.int16), i.view(torch.int16))
    del l, probs, vals, idx
    torch.cuda.empty_cache()
