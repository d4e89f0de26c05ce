"""attn_fwd_workspace with more than 64 query positions on grids of tiles that would leave most of the chip idle, against the
fp64 CPU reference: edges of the 128-row blocks, several heads packed into one, rows that see no key, strided views."""
import numpy as np
import pytest

from paper_2604_18616_amd import inputs as I
from tests._util import check, from_dev_bf16, oracle_parallel, to_dev
from tests.test_attn_split_gpu import call

# B, Hq, Hkv, Sq, Sk, D, causal
SHAPES = [
    (1, 1, 1, 65, 2000, 128, True),
    (1, 2, 1, 130, 1500, 64, False),      # 260 packed rows: three blocks, the last with four rows
    (2, 2, 2, 257, 1029, 128, True),
    (1, 3, 1, 128, 1600, 128, True),      # whole blocks, a head each
    (1, 1, 1, 2000, 1500, 64, True),      # the first 500 rows see no key
    (1, 1, 1, 1100, 1000, 128, True),     # the first 100
]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B%d_H%d_%d_S%d_%d_D%d_%s" % s)
def test_long_queries_against_the_reference(shape):
    from paper_2604_18616_amd import binding
    B, Hq, Hkv, Sq, Sk, D, causal = shape
    assert binding.load_library().attn_fwd_workspace_bytes(B, Hq, Hkv, Sq, Sk, D) > 0
    w = I.Workload("split", B, Hq, Hkv, Sq, Sk, D, causal, 47)
    qb, kb, vb = I.make_qkv(w)
    ref = oracle_parallel(qb, kb, vb, causal, w.scale)
    q, k, v = to_dev(qb), to_dev(kb), to_dev(vb)
    for splits in (0, 2, 7, 33):
        print(shape, splits, flush=True)
        o, lse = call(q, k, v, causal, w.scale, splits)
        check(from_dev_bf16(o), lse.cpu().numpy().astype(np.float64), *ref, "%s splits %d" % (shape, splits))


@pytest.mark.gpu
def test_strided_views_through_the_binding():
    import torch
    from paper_2604_18616_amd import attn_fwd, binding
    gen = torch.Generator(device="cuda").manual_seed(48)
    B, Hq, Hkv, Sq, Sk, D = 2, 4, 2, 200, 1900, 128
    assert binding.load_library().attn_fwd_workspace_bytes(B, Hq, Hkv, Sq, Sk, D) > 0
    rows = lambda h, s, n: torch.randn((B, n, h, D), generator=gen, device="cuda", dtype=torch.bfloat16)[:, :s].transpose(1, 2)
    q, k, v = rows(Hq, Sq, Sq), rows(Hkv, Sk, 2048), rows(Hkv, Sk, 2048)
    o, lse = attn_fwd(q, k, v, causal=True)
    want = attn_fwd(q.contiguous(), k.contiguous(), v.contiguous(), causal=True)
    assert torch.equal(o.contiguous(), want[0]) and torch.equal(lse, want[1])


def test_which_calls_are_cut():
    from paper_2604_18616_amd import binding
    need = binding.load_library().attn_fwd_workspace_bytes
    for shape in [(1, 1, 1, 2048, 18000, 128), (2, 32, 8, 128, 5000, 128), (1, 16, 16, 512, 2500, 128)]:
        assert need(*shape) > 0, shape
    # a full grid, a grid with most of the chip at work, few keys, invalid sizes
    for shape in [(4, 32, 8, 4096, 4096, 128), (2, 32, 8, 512, 5000, 128), (8, 32, 8, 100, 2000, 128), (1, 8, 1, 65, 300, 128), (1, 8, 1, 0, 300, 128), (1, 8, 1, 200, 5000, 96)]:
        assert need(*shape) == 0, shape
