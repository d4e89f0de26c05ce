"""attn_fwd_workspace (few query rows, keys cut over workgroups) against the fp64 CPU reference, at the edges of its cuts:
one tile per key group and one key more or less, 1 / 32 / 33 / 64 / 65 packed query rows, empty parts, both combine
kernels, and the call without memory."""
import numpy as np
import pytest

from paper_2604_18616_amd import inputs as I
from tests._util import check, from_dev_bf16, oracle_parallel, to_dev

pytestmark = pytest.mark.gpu

# B, Hq, Hkv, Sq, Sk, D, causal
SHAPES = [
    (1, 2, 2, 1, 129, 128, False),       # 5 tiles, the last with one key
    (2, 8, 1, 4, 1000, 128, True),       # 32 packed rows: one row block
    (1, 3, 1, 11, 417, 64, True),        # 33: two row blocks share a workgroup's tiles
    (2, 2, 1, 32, 640, 128, True),       # 64
    (1, 5, 1, 13, 333, 128, False),      # 65: four row blocks
    (1, 6, 2, 64, 161, 64, True),        # 192 rows: two workgroups along the rows
    (1, 1, 1, 1, 8300, 64, False),       # 130 parts of two tiles and empty ones, where 256 are asked for
    (1, 2, 1, 1, 16500, 64, False),      # 172 of three
    (1, 1, 1, 2, 33000, 128, False),     # 207 of five
    (1, 8, 1, 4, 60000, 128, True),      # 157 parts of 12 tiles: the library's own cut is that fine
    (128, 8, 8, 1, 1000, 64, False),     # D = 64, two wavefronts per workgroup
]


def call(q, k, v, causal, scale, splits, memory=True, lse=True):
    import torch
    from paper_2604_18616_amd import binding
    lib = binding.load_library()
    B, Hq, Sq, D = q.shape
    o = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    ls = torch.full(q.shape[:3], float("nan"), dtype=torch.float32, device="cuda")
    n = 4 * B * Hq * Sq * max(splits, 1) * (D + 2) if splits else lib.attn_fwd_workspace_bytes(B, Hq, k.shape[1], Sq, k.shape[2], D)
    ws = torch.full((max(n, 16),), 0xFF, dtype=torch.uint8, device="cuda")
    s3 = binding._strides3
    rc = lib.attn_fwd_workspace(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), ls.data_ptr() if lse else None,
                                B, Hq, k.shape[1], Sq, k.shape[2], D, s3(q), s3(k), s3(v), s3(o), int(causal), scale,
                                ws.data_ptr() if memory else None, n if memory else 0, splits,
                                torch.cuda.current_stream().cuda_stream)
    assert rc == 0, binding.strerror(rc)
    torch.cuda.synchronize()
    # the parts that ran: a cut call writes all of the memory it asks for, the surplus parts as empty ones; an uncut call none
    cut = memory and (splits > 1 if splits else n > 0)
    left = ws.view(torch.int32) == -1
    assert not bool(left.any()) if cut else bool(left.all()), (q.shape, k.shape, splits)
    return o, ls


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B%d_H%d_%d_S%d_%d_D%d_%s" % s)
def test_every_cut_against_the_reference(shape):
    B, Hq, Hkv, Sq, Sk, D, causal = shape
    w = I.Workload("split", B, Hq, Hkv, Sq, Sk, D, causal, 41)
    qb, kb, vb = I.make_qkv(w)
    ref = oracle_parallel(qb, kb, vb, causal, w.scale)
    q, k, v = to_dev(qb), to_dev(kb), to_dev(vb)
    for splits in (0, 1, 2, 5, 8, 9, 64, 65, 256):
        print(shape, splits, flush=True)
        o, lse = call(q, k, v, causal, w.scale, splits)
        check(from_dev_bf16(o), lse.cpu().numpy().astype(np.float64), *ref, "%s splits %d" % (shape, splits))
    # without memory: uncut
    o1, lse1 = call(q, k, v, causal, w.scale, 1)
    o0, lse0 = call(q, k, v, causal, w.scale, 7, memory=False)
    assert bool((o0 == o1).all()) and bool((lse0 == lse1).all())
    o2, _ = call(q, k, v, causal, w.scale, 3, lse=False)
    assert np.abs(from_dev_bf16(o2) - ref[0]).max() <= 2e-2


@pytest.mark.parametrize("direction", ["rising", "falling"])
@pytest.mark.parametrize("splits", [1, 6, 40])
def test_score_maxima_that_differ_between_the_parts(direction, splits):
    """Keys scaled along the sequence: every key group and every part has its own maximum, far from the others'."""
    w = I.Workload("drift", 1, 4, 2, 3, 900, 128, False, 42)
    qb, kb, vb = I.make_qkv(w)
    k32 = I.bf16_bits_to_f32(kb)
    ramp = np.linspace(0.0, 12.0, w.Sk, dtype=np.float32)[None, None, :, None]
    kb = I.f32_to_bf16_bits(k32 * (ramp if direction == "rising" else ramp[:, :, ::-1]))
    ref = oracle_parallel(qb, kb, vb, w.causal, w.scale)
    o, lse = call(to_dev(qb), to_dev(kb), to_dev(vb), w.causal, w.scale, splits)
    check(from_dev_bf16(o), lse.cpu().numpy().astype(np.float64), *ref, direction)


def test_keys_past_the_last_one_are_not_read_into_the_result():
    """K and V are the first rows of longer buffers whose other rows hold NaN."""
    import torch
    from paper_2604_18616_amd import attn_fwd
    gen = torch.Generator(device="cuda").manual_seed(43)
    full = lambda: torch.full((2, 512, 4, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    q = torch.randn((2, 2, 8, 128), generator=gen, device="cuda", dtype=torch.bfloat16).transpose(1, 2)
    k, v = full(), full()
    for t in (k, v):
        t[:, :301] = torch.randn((2, 301, 4, 128), generator=gen, device="cuda", dtype=torch.bfloat16)
    k, v = (t[:, :301].transpose(1, 2) for t in (k, v))
    o, lse = attn_fwd(q, k, v, causal=True)
    want = attn_fwd(q.contiguous(), k.contiguous(), v.contiguous(), causal=True)
    assert torch.isfinite(o.float()).all() and torch.equal(o.contiguous(), want[0]) and torch.equal(lse, want[1])


def test_call_on_another_stream_than_torchs_current_one():
    import torch
    from paper_2604_18616_amd import attn_fwd
    gen = torch.Generator(device="cuda").manual_seed(44)
    q, k, v = (torch.randn((1, 4, s, 64), generator=gen, device="cuda", dtype=torch.bfloat16) for s in (1, 3000, 3000))
    want = attn_fwd(q, k, v)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    got = attn_fwd(q, k, v, stream=side)
    torch.cuda.synchronize()
    assert (got[0].float() - want[0].float()).abs().max() <= 2e-2 and (got[1] - want[1]).abs().max() <= 1e-3


# B, Hq, Hkv, Sq, Sk, D: one to five heads on a kv head, one, two and four row blocks per workgroup
@pytest.mark.parametrize("shape", [(2, 4, 2, 64, 400, 128), (1, 2, 1, 64, 449, 64), (1, 3, 3, 40, 513, 128), (1, 6, 2, 50, 513, 64), (1, 5, 1, 33, 513, 128), (1, 2, 1, 200, 1900, 128)],
                         ids=lambda s: "B%d_H%d_%d_S%d_%d_D%d" % s)
@pytest.mark.parametrize("splits", [1, 3])
def test_values_behind_the_mask_reach_no_row_from_further_away_than_in_the_tiled_kernels(shape, splits):
    """V holds infinities and NaN at the last key.  The tiled kernels multiply 0 by them in the 64-key tile in which the
    last of a group of 32 query positions ends, and nowhere before it; nor may the cut do so."""
    B, Hq, Hkv, Sq, Sk, D = shape
    w = I.Workload("mask", B, Hq, Hkv, Sq, Sk, D, True, 45)
    qb, kb, vb = I.make_qkv(w)
    vb[:, :, -1] = 0
    o_ref, lse_ref = oracle_parallel(qb, kb, vb, True, w.scale)
    bad = vb.copy()
    bad[:, :, -1, ::2], bad[:, :, -1, 1::2] = 0x7F80, 0x7FC0
    print(shape, splits, flush=True)
    o, lse = call(to_dev(qb), to_dev(kb), to_dev(bad), True, w.scale, splits)
    o, lse = from_dev_bf16(o), lse.cpu().numpy().astype(np.float64)
    last = (Sk - Sq) + np.minimum(np.arange(Sq) // 32 * 32 + 31, Sq - 1)
    clean = last // 64 * 64 + 63 < Sk - 1
    assert clean.any()
    check(o[:, :, clean], lse[:, :, clean], o_ref[:, :, clean], lse_ref[:, :, clean], str(shape))
    assert not np.isfinite(o[:, :, -1]).any() and np.abs(lse - lse_ref).max() <= 1e-3     # the last row sees the key


@pytest.mark.parametrize("splits", [1, 2])
def test_a_score_that_is_no_number_shows_in_o_and_lse(splits):
    """The last key, alone in its tile, is NaN: every row that sees it gives NaN, and no finite LSE, as the 128-row kernel does."""
    from tests._util import run_hip
    w = I.Workload("nan", 1, 4, 2, 3, 129, 128, False, 46)
    qb, kb, vb = I.make_qkv(w)
    kb[:, :, -1] = 0x7FC0
    o, lse = call(to_dev(qb), to_dev(kb), to_dev(vb), False, w.scale, splits)
    want = run_hip(qb, kb, vb, False, w.scale, wg_rows=128)
    assert np.isnan(from_dev_bf16(o)).all() and np.isnan(want[0]).all()
    assert np.array_equal(lse.cpu().numpy().astype(np.float64), want[1])


def test_results_repeat_exactly():
    import torch
    from paper_2604_18616_amd import attn_fwd
    gen = torch.Generator(device="cuda").manual_seed(47)
    q, k, v = (torch.randn((2, h, s, 128), generator=gen, device="cuda", dtype=torch.bfloat16) for h, s in ((8, 4), (2, 3000), (2, 3000)))
    first = attn_fwd(q, k, v, causal=True)
    for _ in range(5):
        again = attn_fwd(q, k, v, causal=True)
        assert torch.equal(again[0], first[0]) and torch.equal(again[1], first[1])


# B, Hq, Hkv, Sq, Sk, D, causal: more than 64 packed rows on a kv head and few heads, without memory and where no cut pays
@pytest.mark.parametrize("shape,cut", [((1, 8, 1, 32, 1500, 128, True), True), ((7, 8, 2, 52, 800, 64, False), True), ((5, 16, 2, 50, 296, 64, True), False),
                                       ((3, 16, 2, 15, 170, 128, False), False), ((25, 8, 2, 20, 238, 128, False), False)],
                         ids=lambda s: "B%d_H%d_%d_S%d_%d_D%d_%s" % s if isinstance(s, tuple) else "cut" if s else "uncut")
def test_uncut_calls_of_many_packed_rows_run_on_the_128_row_kernel(shape, cut):
    """One workgroup along the keys is slower there than the 128-row kernel's workgroup per head: the same bits as attn_fwd_tile."""
    from paper_2604_18616_amd import binding
    from tests._util import run_hip
    B, Hq, Hkv, Sq, Sk, D, causal = shape
    assert (binding.load_library().attn_fwd_workspace_bytes(B, Hq, Hkv, Sq, Sk, D) > 0) == cut
    w = I.Workload("rows", B, Hq, Hkv, Sq, Sk, D, causal, 48)
    qb, kb, vb = I.make_qkv(w)
    want = run_hip(qb, kb, vb, causal, w.scale, wg_rows=128)
    got = run_hip(qb, kb, vb, causal, w.scale)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    for splits, memory in ((1, True), (7, False)) + (() if cut else ((0, True),)):
        o, lse = call(to_dev(qb), to_dev(kb), to_dev(vb), causal, w.scale, splits, memory=memory)
        assert np.array_equal(from_dev_bf16(o), want[0]) and np.array_equal(lse.cpu().numpy().astype(np.float64), want[1])


def test_four_row_blocks_per_workgroup_uncut():
    """More heads than the 128-row kernel has places for: the kernel of the cut, uncut."""
    w = I.Workload("rows", 16, 36, 4, 8, 130, 128, True, 49)      # 72 packed rows, 576 heads
    qb, kb, vb = I.make_qkv(w)
    o, lse = call(to_dev(qb), to_dev(kb), to_dev(vb), True, w.scale, 1)
    check(from_dev_bf16(o), lse.cpu().numpy().astype(np.float64), *oracle_parallel(qb, kb, vb, True, w.scale), "uncut")
