"""The expert products' pipeline at its edges: row scales are loaded by fours, weights up to three stages ahead.  One to nine
128-deep stages on the codes of 64 to 160 rows, four to nine on those of 192 to 256, whose call has to be large enough for them;
with a workgroup per CU at most and with more of them, whole and half column tiles of the down product.  (One to three stages
of the large codes: test_moe_tiles_gpu; of 32 rows: test_moe_few_gpu.)"""
import pytest

from paper_2604_18616_amd import binding
from tests.test_moe_tiles_gpu import check_rows_per_expert, tiles_256

pytestmark = pytest.mark.gpu

COUNTS = (17, 65, 129, 161, 193, 225, 256)


# too few workgroups for the larger tiles: cut into 128 rows
@pytest.mark.parametrize("H,Isz", [(128, 128), (256, 384), (512, 640), (640, 512), (896, 1152)])
@pytest.mark.parametrize("many", [False, True])
def test_stage_counts(H, Isz, many):
    filler = (40,) * (129 if many else 0)
    rt = binding.load_library().moe_ffn_fp8_row_tiles
    check_rows_per_expert(COUNTS, H, Isz, filler=filler, tiles=sum(rt(n, 128) for n in COUNTS + filler))


# gate/up stages and workgroups, down stages and wide column tiles: 5, 428, 4, 321; 7, 243, 9, 108 (taken by halves); 7, 603, 9, 268;
# 9, 235, 5, 235
@pytest.mark.parametrize("H,Isz,more", [(640, 512, 100), (896, 1152, 20), (896, 1152, 60), (1152, 640, 40)])
def test_stage_counts_of_large_tiles(H, Isz, more):
    filler = (256,) * more
    check_rows_per_expert(COUNTS, H, Isz, filler=filler, tiles=tiles_256(COUNTS + filler))
