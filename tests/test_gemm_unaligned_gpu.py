"""gemm_bf16 on operands that are not 16-byte aligned, against the fp64 reference with the tolerance of
test_gemm_parity_gpu: one stage along k and a fraction more, an overlap of all but one element, one tile along n and a
fraction more, single rows, pitches and pointers that are odd, all three tiles (for B stored [K,N] the 128 x 128 one from 128
columns on) and both storages of B."""
import numpy as np
import pytest

from paper_2604_18616_amd import inputs as I
from tests.test_gemm_parity_gpu import check_full, run

pytestmark = pytest.mark.gpu

# M, N, K, extra columns of (a, b, c), element offset of every pointer
CASES = [(1, 64, 64, (0, 1, 0), 1), (33, 65, 65, (0, 0, 0), 0), (64, 127, 127, (0, 0, 0), 0), (65, 129, 128, (1, 0, 0), 0), (130, 200, 191, (3, 5, 1), 3),
         (257, 191, 320, (8, 0, 8), 1), (7, 77, 1000, (0, 0, 0), 0), (129, 385, 577, (0, 0, 2), 5), (96, 33, 201, (0, 0, 0), 0)]


@pytest.mark.parametrize("tile", [64, 128, 1284, 0])
@pytest.mark.parametrize("b_is_nk", [False, True])
@pytest.mark.parametrize("M,N,K,pad,shift", CASES)
def test_unaligned_rows(M, N, K, pad, shift, b_is_nk, tile):
    check_full(M, N, K, b_is_nk, seed=700 + M + N + K, pad=pad, shift=shift, tile=tile)


@pytest.mark.parametrize("b_is_nk", [False, True])
def test_infinities_stay_where_the_definition_puts_them(b_is_nk):
    """The stage at the end of k re-reads elements the stage before it has used: an infinity among them must not
    turn into 0 * inf."""
    M, N, K = 70, 75, 100
    rng = np.random.default_rng(5)
    A, B = (rng.integers(1, 4, size=s).astype(np.float32) for s in ((M, K), (K, N)))
    A[3, 40] = np.inf                                  # k = 40: seen by the first stage and by the second
    B[50, 7] = -np.inf
    want = A.astype(np.float64) @ B.astype(np.float64)
    for tile in (64, 128, 1284):
        got = run(I.f32_to_bf16_bits(A), I.f32_to_bf16_bits(np.ascontiguousarray(B.T) if b_is_nk else B), b_is_nk, tile=tile)
        finite = np.isfinite(want)
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(got[~finite & ~np.isnan(want)], want[~finite & ~np.isnan(want)])
        assert np.all(np.abs(got[finite] - want[finite]) <= 2.0 ** -8 * want[finite])
