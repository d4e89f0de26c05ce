"""moe_ffn_fp8 with few rows per expert: two workgroups per CU with tiles of 32 rows.  Taken with up to 32 tokens and 12 slots per
expert, or up to 64 tokens and 4 slots per expert; on either side of both lines, and with an expert favoured beyond one tile."""
import numpy as np
import pytest

import oracle
from paper_2604_18616_amd import inputs as I
from tests.test_moe_parity_gpu import check_routing, check_stage1, check_y, run, sanity_net
from tests.test_moe_tiles_gpu import check_rows_per_expert


def tiles_32(counts):
    return sum(-(-n // 32) for n in counts)

pytestmark = pytest.mark.gpu


# one and two tiles of 32 rows, 32 and 64 tokens; 128 wide column tiles of the down product and fewer (halved, three
# stages of weights), and more; one to nine 128-deep stages
@pytest.mark.parametrize("counts", [(1,), (12, 3), (31, 1), (32,), (33, 2), (31, 33), (64,)])
@pytest.mark.parametrize("H,Isz,ones", [(128, 128, 0), (640, 384, 16), (384, 1152, 16), (2944, 256, 60), (1152, 640, 60)])
def test_favoured_experts(counts, H, Isz, ones):
    ones = min(ones, (32 if sum(counts) <= 32 and ones < 60 else 64) - sum(counts))
    tokens = sum(counts) + ones
    per = 12 if tokens <= 32 else 4
    filler = (1,) * ones + (0,) * max(0, -(-tokens // per) - len(counts) - ones)
    check_rows_per_expert(counts, H, Isz, filler=filler, tiles=tiles_32(counts + filler))


# one token or one expert to the other side of each line: the general kernel, whose tiles a favoured expert does not outgrow
@pytest.mark.parametrize("counts,filler", [((33,), (0,) * 7), ((64,), (0,) * 14), ((64,), (1,) + (0,) * 20), ((20, 12), ())])
def test_beyond_the_lines(counts, filler):
    check_rows_per_expert(counts, 640, 384, filler=filler)


@pytest.mark.parametrize("counts,filler", [((10, 12), (1,) * 8), ((33,), (1,) * 10 + (0,) * 12)])
def test_two_local_slots(counts, filler):
    check_rows_per_expert(counts, 256, 256, twice=True, filler=filler)


# nothing says that a token's choices differ: all slots on one expert, or all but one
@pytest.mark.parametrize("T,KTOP,E,others", [(64, 4, 64, 0), (32, 16, 43, 0), (64, 4, 64, 1), (1, 12, 1, 0)])
def test_repeated_choices(T, KTOP, E, others):
    w = I.MoeWorkload("t", T, 77 + T + others, H=384, I=640, E=E, KTOP=KTOP, EP=1)
    d = I.make_moe(w)
    ids = np.full((T, KTOP), E - 1, np.int32)
    ids[:, :others] = 0
    d["ids"] = ids
    print("repeated choices", T, KTOP, E, others, flush=True)
    g = run(d)
    assert g["ntiles"] == tiles_32((T * others, T * (KTOP - others)))
    check_routing(w, d, g)
    check_stage1(w, d, g, [0, T - 1])
    check_y(w, d, g, sorted({0, T // 2, T - 1}))
    sanity_net(g["y"], oracle.moe_ref(**d), "repeated")
