"""The expert products' pipeline at its edges: one to nine 128-deep stages (row scales are loaded by fours, weights up to three
stages ahead), for every tile size, with a workgroup per CU at most and with more of them."""
import pytest

from tests.test_moe_tiles_gpu import check_rows_per_expert

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Isz", [(128, 128), (256, 384), (512, 640), (640, 512), (896, 1152)])
@pytest.mark.parametrize("many", [False, True])
def test_stage_counts(H, Isz, many):
    check_rows_per_expert((17, 65, 129, 161, 193, 225, 256), H, Isz, filler=(40,) * (129 if many else 0))
