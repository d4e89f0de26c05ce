"""attn_fwd with few keys, where workgroups have 128 or 256 rows by an estimate (D = 128; up to 512 keys, causal up to 352 visible
to a row in the mean), and just beyond: both are taken here."""
import pytest
import torch

from paper_2604_18616_amd import attn_fwd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Sq,Sk", [(128, 128), (300, 511), (512, 512), (513, 513), (700, 513), (704, 704), (705, 705), (65, 352), (900, 600)])
@pytest.mark.parametrize("causal", [False, True])
def test_few_keys(Sq, Sk, causal):
    torch.manual_seed(Sq + Sk)
    B, Hq, Hkv, D = 17, 16, 2, 128                         # more than 128 workgroups of 256 rows
    q, k, v = (torch.randn(B, h, s, D, device="cuda", dtype=torch.bfloat16) for h, s in ((Hq, Sq), (Hkv, Sk), (Hkv, Sk)))
    print("few keys", Sq, Sk, causal, flush=True)
    o, lse = attn_fwd(q, k, v, causal=causal)
    b, heads = 13, [3, 12]
    s = torch.stack([q[b, h].double() @ k[b, h // 8].double().t().contiguous() for h in heads]) * D ** -0.5
    if causal:
        hidden = torch.arange(Sk, device="cuda")[None] > torch.arange(Sq, device="cuda")[:, None] + (Sk - Sq)
        s.masked_fill_(hidden, float("-inf"))
    want_lse = torch.logsumexp(s, dim=2)
    p = torch.where(want_lse[..., None] == float("-inf"), torch.zeros_like(s), (s - want_lse[..., None]).exp())
    want = torch.stack([p[i] @ v[b, h // 8].double() for i, h in enumerate(heads)])
    # one rounding of O and of every probability to bf16: 2^-9 of the largest |V| that enters each
    assert (o[b, heads].double() - want).abs().max() <= 2 ** -8 * v.abs().max()
    assert torch.equal(lse[b, heads] == float("-inf"), want_lse == float("-inf"))
    seen = want_lse > float("-inf")
    assert (lse[b, heads].double() - want_lse)[seen].abs().max() <= 1e-4
    assert torch.isfinite(o).all()
