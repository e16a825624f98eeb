"""GPU parity: slimfit_prune_global / slimfit_restore_global (Alg. 5 on the whole flattened
tensor) vs the CPU oracle.  Values and indices must be bit-identical."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2305_18513_amd import binding as sf
from paper_2305_18513_amd import synth
from tests.gpu_util import Guarded, require_gpu, to_np

pytestmark = pytest.mark.gpu


def _bits(a):
    return a.view(np.uint32) if a.dtype == np.float32 else a


def _run_both(x: torch.Tensor, k: int, by_magnitude: bool, restore=True, workspace=None):
    n = x.numel()
    vals = Guarded(k, x.dtype)
    idx = Guarded(k, torch.int32)
    ws = Guarded(sf.prune_global_workspace(n), torch.uint8) if workspace is None else workspace
    ptr = Guarded(sf.global_tile_ptr_len(n), torch.int32)
    sf.prune_global(x, k, vals.t, idx.t, by_magnitude=by_magnitude, tile_ptr=ptr.t, workspace=ws.t)
    torch.cuda.synchronize()
    vals.check(); idx.check(); ws.check(); ptr.check()
    ov, oi = ref.prune_global(to_np(x), k, by_magnitude=by_magnitude)
    np.testing.assert_array_equal(to_np(idx.t), oi)
    np.testing.assert_array_equal(_bits(to_np(vals.t)), _bits(ov))
    # tile pointers: survivors ahead of every 4096 elements, counted on the oracle's index list
    edges = np.arange(ptr.t.numel(), dtype=np.int64) * sf.GLOBAL_TILE
    np.testing.assert_array_equal(to_np(ptr.t), np.searchsorted(oi, edges, side="left").astype(np.int32))
    assert int(ptr.t[-1]) == k
    if restore:
        want = _bits(ref.restore_global(ov, oi, n))
        for tp in (None, ptr.t):                                   # zeros + scatter, and the one-pass form
            out = Guarded(n, x.dtype)
            sf.restore_global(vals.t, idx.t, k, out.t, tile_ptr=tp)
            torch.cuda.synchronize()
            out.check()
            np.testing.assert_array_equal(_bits(to_np(out.t)), want)
    # the pointer list is optional
    vals2 = Guarded(k, x.dtype)
    idx2 = Guarded(k, torch.int32)
    sf.prune_global(x, k, vals2.t, idx2.t, by_magnitude=by_magnitude, workspace=ws.t)
    torch.cuda.synchronize()
    vals2.check(); idx2.check()
    assert torch.equal(idx2.t, idx.t) and torch.equal(vals2.t.view(torch.uint8), vals.t.view(torch.uint8))
    return oi


SIZES = [(1, 1), (5, 2), (63, 63), (64, 6), (4096, 409), (4097, 1), (4097, 4097), (10000, 1000),
         (70001, 7000), (8192 * 3 + 5, 2500), ((1 << 20) + 3, 104857)]


@pytest.mark.parametrize("by_mag", [True, False])
@pytest.mark.parametrize("n,k", SIZES)
def test_fp32_random_ties_and_constant(n, k, by_mag):
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(n * 3 + k)
    x = torch.randn(n, generator=g, device="cuda")
    _run_both(x, k, by_mag)
    _run_both((x * 2).round() / 2, k, by_mag)                       # heavy ties, both signs, +-0
    _run_both(torch.full((n,), -0.75, device="cuda"), k, by_mag)    # every key equal
    z = torch.zeros(n, device="cuda")
    z[::2] = -0.0
    _run_both(z, k, by_mag)


@pytest.mark.parametrize("by_mag", [True, False])
@pytest.mark.parametrize("n,k", SIZES)
def test_bf16_random_ties_and_constant(n, k, by_mag):
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(n * 5 + k)
    x = torch.randn(n, generator=g, device="cuda").bfloat16()
    _run_both(x, k, by_mag)
    _run_both(((x.float() * 2).round() / 2).bfloat16(), k, by_mag)
    _run_both(torch.full((n,), -0.75, device="cuda").bfloat16(), k, by_mag)


def test_wide_dynamic_range_and_infinities():
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(11)
    n = 50000
    x = torch.randn(n, generator=g, device="cuda") * torch.exp2(torch.randint(-120, 120, (n,), generator=g,
                                                                              device="cuda").float())
    x[17] = float("inf")
    x[4099] = float("-inf")
    x[33] = 1e-42                                                     # subnormal
    x[34] = -1e-42
    for k in (1, 2, 3, 5000, n - 1):
        _run_both(x, k, True, restore=False)
        _run_both(x, k, False, restore=False)


def test_bunched_candidates_overflow_a_sub_list():
    """The keys that share the cut's leading digit sit in one tile: the candidate list gives up and the
    digits are counted from the tensor instead."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(21)
    n = 1 << 21
    for dtype in (torch.float32, torch.bfloat16):
        x = torch.rand(n, generator=g, device="cuda") * 0.5
        x[1000:4000] = 1.0 + torch.rand(3000, generator=g, device="cuda") * 0.06      # one 1/16-binade bin
        hot = torch.randperm(n, generator=g, device="cuda")[:100]
        hot = hot[(hot < 1000) | (hot >= 4000)]
        x[hot] = 2.0 + torch.rand(hot.numel(), generator=g, device="cuda")
        x = (x * torch.where(torch.rand(n, generator=g, device="cuda") < 0.5, -1.0, 1.0)).to(dtype)
        _run_both(x, int(hot.numel()) + 1500, True)
        # the same keys spread over the tensor take the list
        _run_both(x[torch.randperm(n, generator=g, device="cuda")].contiguous(), int(hot.numel()) + 1500, True)


def test_workspace_is_reusable_and_need_not_be_clean():
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(5)
    ws = Guarded(sf.prune_global_workspace(100000), torch.uint8)     # starts as 0xAB bytes
    for n, k in ((100000, 10000), (9000, 17), (100000, 99999)):
        x = torch.randn(n, generator=g, device="cuda")
        _run_both(x, k, True, workspace=ws)


def test_k_zero_and_empty_are_no_ops():
    require_gpu()
    x = torch.randn(100, device="cuda")
    vals = Guarded(4, torch.float32)
    idx = Guarded(4, torch.int32)
    before = vals.raw.clone()
    sf.prune_global(x, 0, vals.t, idx.t)
    sf.prune_global(x[:0], 0, vals.t, idx.t)
    torch.cuda.synchronize()
    assert torch.equal(before, vals.raw)
    out = Guarded(100, torch.float32)
    sf.restore_global(vals.t, idx.t, 0, out.t)
    torch.cuda.synchronize()
    out.check()
    assert not out.t.any()


def test_restore_skips_bad_indices_and_accepts_any_order():
    require_gpu()
    vals = torch.tensor([1.0, 2.0, 3.0, 4.0], device="cuda")
    idx = torch.tensor([7, -1, 0, 12], dtype=torch.int32, device="cuda")
    out = Guarded(9, torch.float32)
    sf.restore_global(vals, idx, 4, out.t)
    torch.cuda.synchronize()
    out.check()
    assert out.t.tolist() == [3.0, 0, 0, 0, 0, 0, 0, 1.0, 0]


def test_restore_with_inconsistent_tile_pointers_stays_in_bounds():
    require_gpu()
    n, k = 10000, 6
    vals = torch.arange(1, k + 1, device="cuda").float()
    idx = torch.tensor([5, 4095, 4096, 9000, 9999, 123456], dtype=torch.int32, device="cuda")
    out = Guarded(n, torch.float32)
    good = torch.tensor([0, 2, 3, 6], dtype=torch.int32, device="cuda")
    sf.restore_global(vals, idx, k, out.t, tile_ptr=good)
    torch.cuda.synchronize()
    out.check()
    want = torch.zeros(n)
    want[[5, 4095, 4096, 9000, 9999]] = torch.tensor([1.0, 2.0, 3.0, 4.0, 5.0])
    assert torch.equal(out.t.cpu(), want)
    for bad in ([0, 6, 6, 6], [-5, 100, 3, 99], [6, 0, 0, 0], [0, 0, 0, 0]):
        sf.restore_global(vals, idx, k, out.t, tile_ptr=torch.tensor(bad, dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        out.check()
        got = out.t.cpu()
        assert bool(((got == 0) | (got == want)).all())            # misplaced pairs are dropped, nothing else appears


def test_argument_errors():
    require_gpu()
    x = torch.randn(4096, device="cuda")
    vals = torch.empty(16, device="cuda")
    idx = torch.empty(16, dtype=torch.int32, device="cuda")
    ws = torch.empty(sf.prune_global_workspace(4096), dtype=torch.uint8, device="cuda")
    cases = [
        (dict(x=x, k=5000), sf.ERR_INVALID_ARG),                      # k > n
        (dict(x=x, k=-1), sf.ERR_INVALID_ARG),
        (dict(x=x[1:], k=4), sf.ERR_ALIGNMENT),
        (dict(x=x, k=4, workspace=ws[:64]), sf.ERR_WORKSPACE),
    ]
    for kw, want in cases:
        kw.setdefault("workspace", ws)
        xx = kw.pop("x")
        k = kw.pop("k")
        with pytest.raises(sf.SlimfitError) as e:
            sf.prune_global(xx, k, vals if k <= 16 else torch.empty(max(k, 1), device="cuda"),
                            idx if k <= 16 else torch.empty(max(k, 1), dtype=torch.int32, device="cuda"), **kw)
        assert e.value.status == want
    with pytest.raises(sf.SlimfitError):
        sf.prune_global_workspace(1 << 31)


@pytest.mark.parametrize("ci", [1, 2, 3, 4])
def test_layernorm_input_at_full_size(ci):
    """The paper's placement: 10 % of the standardised LayerNorm input, whole batch."""
    require_gpu()
    cfg = synth.CONFIGS[ci]
    x = synth.activation(cfg, "ln_in", device="cuda").reshape(-1)
    k = sf.keep_count(x.numel(), 100000)
    assert k == int(x.numel() * 0.1)
    _run_both(x, k, True)


# ---- sizes past the sample (65 536 entries) and the edges of the record route ----

def _signs(g, n):
    return torch.where(torch.rand(n, generator=g, device="cuda") < 0.5, -1.0, 1.0)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,k", [(200003, 200003 // 9), (200003, 200003 // 9 + 1), (300000, 1), (300001, 299999), (300001, 700),
                                 (1 << 19, 1 << 18), ((1 << 19) + 4095, 52428)])
def test_records_and_sample_rule(n, k, dtype):
    """One entry in nine is where records stop; ranks near either end take the tensor's own first digit."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(n + k)
    x = torch.randn(n, generator=g, device="cuda").to(dtype)
    _run_both(x, k, True, restore=False)
    _run_both(x, k, False, restore=False)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_tiles_with_more_candidates_than_records(dtype):
    """Two tiles are all candidates (read from the tensor again), the others hold hardly any; then one in which a
    single tile's keys crowd the bracket."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(31)
    n = 40 * 4096 + 77
    x = torch.rand(n, generator=g, device="cuda") * 0.5
    x[3 * 4096:4 * 4096] += 4.0
    x[-3000:] += 2.0
    x = (x * _signs(g, n)).to(dtype)
    for k in (4096 + 1500, 4096 + 3000, 4096 + 3000 + 9000):
        _run_both(x, k, True, restore=False)
    x = torch.exp2(torch.rand(n, generator=g, device="cuda") * 60 - 50)          # many binades wide
    _run_both((x * _signs(g, n)).to(dtype), n // 10, True, restore=False)


def _sampled_vectors(n, epv):
    """The vectors the bracket is estimated from: one of each of 16 384 stretches, at a hashed place."""
    vectors, total = n // epv, 16384
    i = np.arange(total, dtype=np.uint64)
    step = np.uint64((vectors << 16) // total)
    v0, v1 = (i * step) >> np.uint64(16), ((i + np.uint64(1)) * step) >> np.uint64(16)
    h = (i * np.uint64(0x9E3779B1)) & np.uint64(0xFFFFFFFF)
    h ^= h >> np.uint64(15)
    h = (h * np.uint64(0x85EBCA77)) & np.uint64(0xFFFFFFFF)
    h ^= h >> np.uint64(13)
    return (v0 + ((h * (v1 - v0)) >> np.uint64(32))).astype(np.int64)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("scale", [0.25, 4.0])
def test_sample_that_misses_the_cut(dtype, scale):
    """Every entry the sample sees is four times smaller (larger) than the rest: T lies above (below) the bracket, and
    the plain route is taken (word 6 of the workspace), or the sample is no longer where this test thinks it is."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(41)
    epv = 4 if dtype == torch.float32 else 8
    n = 70000 * epv + 3
    x = torch.randn(n, generator=g, device="cuda")
    at = torch.from_numpy((_sampled_vectors(n, epv)[:, None] * epv + np.arange(epv)).reshape(-1)).cuda()
    x[at] *= scale
    x = x.to(dtype)
    for k in (n // 10, n // 2):
        for by_mag in (True, False):
            ws = Guarded(sf.prune_global_workspace(n), torch.uint8)
            _run_both(x, k, by_mag, restore=False, workspace=ws)
            assert int(ws.t[24:28].view(torch.int32)) == 1, (k, by_mag)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("spread", [0.3, 1.0])
@pytest.mark.parametrize("rows,H", [(256, 128), (512, 128), (512, 256), (1024, 512), (2048, 256), (128, 1024), (4096, 768)])
def test_columns_of_unlike_scale(rows, H, spread, dtype):
    """Rows that are whole multiples of 16, or 2 to 8, of the sample's stretches, with columns of log-normal scales: the
    workgroups' brackets lie together, and no list overflows (word 6 of the workspace: the plain route)."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(rows + H)
    x = torch.randn(rows, H, generator=g, device="cuda") * torch.exp(spread * torch.randn(H, generator=g, device="cuda"))
    ws = Guarded(sf.prune_global_workspace(x.numel()), torch.uint8)
    _run_both(x.view(-1).to(dtype), x.numel() // 10, True, restore=False, workspace=ws)
    assert int(ws.t[24:28].view(torch.int32)) == 0


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("at_vals,at_idx", [(0, 0), (1, 1), (2, 2), (3, 3), (0, 1), (3, 2), (2, 0), (1, 3)])
def test_outputs_at_any_place_in_a_vector(at_vals, at_idx, dtype):
    """Survivors leave as 16-byte vectors where both outputs lie alike: values and indices that begin at every element of one, the
    same and another, with nothing written before or behind them."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(61)
    for n, k in ((200003, 20000), (300001, 30001), (70 * 4096, 28001)):
        x = torch.randn(n, generator=g, device="cuda").to(dtype)
        want_vals, want_idx = torch.empty(k, dtype=dtype, device="cuda"), torch.empty(k, dtype=torch.int32, device="cuda")
        sf.prune_global(x, k, want_vals, want_idx)
        oi = ref.prune_global(to_np(x), k, by_magnitude=True)[1]
        np.testing.assert_array_equal(to_np(want_idx), oi)
        vals, idx = Guarded(at_vals + k, dtype), Guarded(at_idx + k, torch.int32)
        sf.prune_global(x, k, vals.t[at_vals:], idx.t[at_idx:])
        torch.cuda.synchronize()
        vals.check(); idx.check()
        assert bool((vals.raw[: at_vals * dtype.itemsize] == 0xAB).all()) and bool((idx.raw[: at_idx * 4] == 0xAB).all())
        assert torch.equal(idx.t[at_idx:], want_idx) and torch.equal(vals.t[at_vals:], want_vals)


def _keys(x: torch.Tensor, by_magnitude):
    """Larger key, earlier in the order; NaN above the infinities by magnitude, beyond the one of their sign by value."""
    b = to_np(x.float()).view(np.uint32).astype(np.int64)
    if by_magnitude:
        return b & 0x7FFFFFFF
    return np.where(b >> 31 == 1, -(b & 0x7FFFFFFF), b)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("by_mag", [True, False])
@pytest.mark.parametrize("n,positive,negative", [(200003, 0.0, 0.02), (200003, 0.02, 0.02), (200003, 0.0, 0.3), (200003, 0.2, 0.2),
                                                 (40 * 4096 + 77, 0.01, 0.005), (3000, 0.02, 0.1)])
def test_nan_have_their_place(n, positive, negative, by_mag, dtype):
    """NaN of either sign, fewer and more of them than are kept: every slot is written, by the order of the keys."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn(n, generator=g, device="cuda").to(dtype)
    u = torch.rand(n, generator=g, device="cuda")
    bits = x.view(torch.int32 if dtype == torch.float32 else torch.int16)
    some = torch.randint(1, 100, (n,), generator=g, device="cuda").to(bits.dtype)
    base, sign = (0x7FC00000, -(1 << 31)) if dtype == torch.float32 else (0x7FC0, -(1 << 15))
    some = torch.where(some < 60, some, torch.zeros_like(some)) if dtype == torch.float32 else some % 60
    bits[u < positive] = (some + base)[u < positive]
    low = u > 1.0 - negative
    bits[low] = ((some + base) | sign)[low]
    k = n // 10
    vals, idx = Guarded(k, dtype), Guarded(k, torch.int32)
    sf.prune_global(x, k, vals.t, idx.t, by_magnitude=by_mag)
    torch.cuda.synchronize()
    vals.check(); idx.check()
    want = np.sort(np.argsort(-_keys(x, by_mag), kind="stable")[:k])
    np.testing.assert_array_equal(to_np(idx.t), want)
    got, ref_bits = vals.t.view(bits.dtype).cpu().numpy(), bits.cpu().numpy()[want]
    np.testing.assert_array_equal(got, ref_bits)


def test_a_bin_of_more_entries_than_a_sixteenth_of_32_bits():
    """All of 2^28 entries share T's bin and the rank is too close to the top for a sample: the bracket is seen to be too much for
    the lists (word 0 of the workspace), not only once they overflow (word 1)."""
    require_gpu()
    n, k = 1 << 28, 1000
    x = torch.full((n,), 1.5, dtype=torch.bfloat16, device="cuda")
    vals, idx = torch.empty(k, dtype=torch.bfloat16, device="cuda"), torch.empty(k, dtype=torch.int32, device="cuda")
    ws = torch.zeros(sf.prune_global_workspace(n), dtype=torch.uint8, device="cuda")
    sf.prune_global(x, k, vals, idx, by_magnitude=True, workspace=ws)
    assert ws[:8].view(torch.int32).tolist() == [1, 0]
    assert torch.equal(idx, torch.arange(k, dtype=torch.int32, device="cuda")) and bool((vals == 1.5).all())


def _least_workspace(n):
    tiles = (n + sf.GLOBAL_TILE - 1) // sf.GLOBAL_TILE
    return 16512 + 2 * ((8 * tiles + 127) // 128 * 128) + 1024 * (tiles + 1)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,k,room", [(1, 1, 0), (5, 2, 0), (4096, 409, 0), (4097, 4097, 0), (70001, 7000, 0), ((1 << 20) + 3, 104857, 0),
                                      (300000, 30000, 150000), (2000003, 200000, 1000001), (2000003, 1500000, 700000),
                                      (6500003, 650000, 0), (6500003, 5, 0), (6500003, 3000000, 0)])
def test_smaller_workspaces(n, k, room, dtype):
    """From the smallest accepted size up: without lists, with short ones, without records."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(n + k)
    least = _least_workspace(n)
    assert least <= (room or least) < sf.prune_global_workspace(n)
    x = torch.randn(n, generator=g, device="cuda").to(dtype)
    for by_mag in (True, False):
        _run_both(x, k, by_mag, restore=False, workspace=Guarded(room or least, torch.uint8))
    _run_both((x * 2).round() / 2, k, True, restore=False, workspace=Guarded(room or least, torch.uint8))
    vals, idx = torch.empty(k, dtype=dtype, device="cuda"), torch.empty(k, dtype=torch.int32, device="cuda")
    with pytest.raises(sf.SlimfitError) as e:
        sf.prune_global(x, k, vals, idx, True, workspace=torch.empty(least - 1, dtype=torch.uint8, device="cuda"))
    assert e.value.status == sf.ERR_WORKSPACE


def test_smaller_workspaces_hold_what_was_reported_before_there_were_records():
    """The sizes that slimfit_prune_global_workspace used to report."""
    for n, want in ((1, 18816), (4096, 18816), (4097, 19840), (100000, 43648), (6500003, 1668224), (50331648, 12797056)):
        assert _least_workspace(n) == want
