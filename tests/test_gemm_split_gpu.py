"""gemm_bf16_workspace (k cut over workgroups) against the fp64 reference, with the tolerance of test_gemm_parity_gpu: the
fp32 sum has one more rounding per part, which that tolerance's (K/16 + 4) steps cover, as a part is at least 64 deep."""
import numpy as np
import pytest

import oracle
from paper_2604_18616_amd import inputs as I
from tests.test_gemm_parity_gpu import check_full, dev, host, tol

pytestmark = pytest.mark.gpu


def run_split(a_bits, b_bits, b_is_nk, tile, splits, pad, given=None):
    """The C entry with a NaN-filled workspace of just the size it asks for, between guard bytes."""
    import torch
    from paper_2604_18616_amd import binding

    M, K = a_bits.shape
    N = b_bits.shape[0] if b_is_nk else b_bits.shape[1]
    a, b = dev(a_bits), dev(b_bits)
    c = torch.full((M, N + pad), float("nan"), dtype=torch.bfloat16, device="cuda")
    need = 4 * M * N * splits if given is None else given
    ws = torch.full((need // 4 + 64,), float("nan"), dtype=torch.float32, device="cuda")
    rc = binding.load_library().gemm_bf16_workspace(a.data_ptr(), b.data_ptr(), c.data_ptr(), M, N, K, K, b.shape[1], N + pad, int(b_is_nk),
                                                    tile, splits, ws.data_ptr(), need, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0
    assert torch.isnan(ws[need // 4:]).all() and torch.isnan(c[:, N:].float()).all()
    return host(c[:, :N])


# M, N, K, splits: whole tiles, one stage per part, k tails in the last part, cuts that leave parts over, single rows
CASES = [(256, 256, 512, 2, 0), (64, 64, 256, 4, 8), (1, 128, 1024, 16, 0), (70, 200, 840, 3, 16), (257, 264, 1096, 5, 0), (130, 72, 136, 7, 8), (16, 1024, 4096, 12, 0)]


# every tile the entry point takes: the 32x32x16 and the 16x16x32 epilogue of each wavefront tile
@pytest.mark.parametrize("tile", [64, 128, 1284, 256, 2564, 25616, 19216, 256416, 12816, 128416, 6416])
@pytest.mark.parametrize("b_is_nk", [False, True])
@pytest.mark.parametrize("M,N,K,splits,pad", CASES)
def test_parts_add_up(M, N, K, splits, pad, b_is_nk, tile):
    a, b = I.make_ab(I.GemmWorkload("t", M, N, K, 900 + M + N + K, b_is_nk=b_is_nk))
    print("split case", M, N, K, splits, b_is_nk, tile, flush=True)
    c = run_split(a, b, b_is_nk, tile, splits, pad)
    ref, s = oracle.gemm_ref(a, b, b_is_nk=b_is_nk)
    assert (np.abs(c - ref) <= tol(ref, s, K)).all()


def test_too_small_a_workspace_means_no_cut():
    a, b = I.make_ab(I.GemmWorkload("t", 64, 64, 1024, 5, b_is_nk=True))
    assert np.array_equal(run_split(a, b, True, 64, 4, 0, given=4 * 64 * 64 * 4 - 16), run_split(a, b, True, 64, 1, 0))


def test_no_memory_left_for_the_parts_means_no_cut(monkeypatch):
    import torch
    from paper_2604_18616_amd import attn_fwd, binding, gemm_bf16
    gen = torch.Generator(device="cuda").manual_seed(6)
    randn = lambda *s: torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16)
    a, b = randn(16, 4096), randn(512, 4096)
    q, k, v = randn(1, 2, 100, 128), randn(1, 2, 3000, 128), randn(1, 2, 3000, 128)
    cut = gemm_bf16(a, b, b_is_nk=True), attn_fwd(q, k, v)[0]
    monkeypatch.setattr(binding, "_scratch", lambda need, device: None)
    whole = gemm_bf16(a, b, b_is_nk=True), attn_fwd(q, k, v)[0]
    assert torch.equal(whole[0], gemm_bf16(a, b, b_is_nk=True, tile=64))
    for x, y in zip(cut, whole):                          # both within a rounding to bf16 and, for P, one before the sum
        assert (x.float() - y.float()).norm() <= 2.0 ** -7 * y.float().norm()


def test_memory_for_the_parts_is_taken_only_where_the_call_can_be_cut(monkeypatch):
    import torch
    from paper_2604_18616_amd import attn_fwd, binding, gemm_bf16
    asked, scratch = [], binding._scratch
    monkeypatch.setattr(binding, "_scratch", lambda need, device: asked.append(need) or scratch(need, device))
    empty = lambda *s: torch.zeros(s, device="cuda", dtype=torch.bfloat16)
    a, b = empty(16, 4096), empty(512, 4096)
    gemm_bf16(a, b, b_is_nk=True)
    assert len(asked) == 1
    shifted = empty(16 * 4096 + 1)[1:].view(16, 4096)             # a row that starts at an odd element
    odd_pitch = empty(16, 4097)[:, :4096]
    odd_result = empty(16, 513)[:, :512]
    gemm_bf16(shifted, b, b_is_nk=True), gemm_bf16(odd_pitch, b, b_is_nk=True), gemm_bf16(a, b, odd_result, b_is_nk=True)
    gemm_bf16(a, b, b_is_nk=True, tile=64), gemm_bf16(a, b, b_is_nk=True, stream=torch.cuda.Stream())
    assert len(asked) == 1
    q, k = empty(1, 2, 4, 128), empty(1, 2, 3000, 128)
    attn_fwd(q, k, k)
    assert len(asked) == 2
    far = empty(3000, 1 << 20).view(1, 1, 3000, 1 << 20)[..., :128]      # one head of K spans more than 4 GiB
    attn_fwd(q[:, :1], far, k[:, :1]), attn_fwd(q, k, k, stream=torch.cuda.Stream())
    assert len(asked) == 2
    torch.cuda.synchronize()


@pytest.mark.parametrize("M,N,K", [(1, 1024, 2048), (100, 512, 4096), (256, 256, 2056), (512, 512, 4096)])
def test_the_librarys_own_cut(M, N, K):
    from paper_2604_18616_amd import binding
    assert binding.load_library().gemm_bf16_workspace_bytes(M, N, K) > 0
    check_full(M, N, K, True, seed=11)
    check_full(M, N, K, False, seed=12)


def test_which_products_are_not_cut():
    from paper_2604_18616_amd import binding
    need = binding.load_library().gemm_bf16_workspace_bytes
    for M, N, K in [(8192, 8192, 8192), (1024, 1024, 1024), (16, 14336, 4096), (4096, 4096, 256), (999, 2001, 1501), (0, 64, 64), (64, 64, -1)]:
        assert need(M, N, K) == 0
