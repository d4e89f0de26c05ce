"""moe_ffn_fp8 with few rows per expert (at most 12 slots each on average): two workgroups per CU with tiles of 32 rows, and
experts that are favoured beyond one such tile."""
import pytest

from tests.test_moe_tiles_gpu import check_rows_per_expert

pytestmark = pytest.mark.gpu


# one to three tiles of 32 rows inside a row tile, a second row tile; 128 wide column tiles of the down product and fewer
# (halved, three stages), and more
@pytest.mark.parametrize("counts", [(1,), (12, 3), (31, 33, 2), (64, 65, 96, 97), (130, 1)])
@pytest.mark.parametrize("H,Isz,empty", [(128, 128, 16), (640, 384, 40), (2944, 256, 60)])
def test_favoured_experts(counts, H, Isz, empty):
    filler = (0,) * max(0, -(-sum(counts) // 12) - len(counts)) + (1,) * empty
    check_rows_per_expert(counts, H, Isz, filler=filler)


def test_two_local_slots():
    check_rows_per_expert((20, 40), 256, 256, twice=True, filler=(1,) * 30)
