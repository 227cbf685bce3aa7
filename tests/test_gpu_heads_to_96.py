"""Heads of 72 to 96 elements run on six MFMA steps a block, in every tile shape that their sizes take: the same bits as those of the same inputs with zeros
added up to 128 elements, on eight (a step of zeros adds nothing)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# (form as krul_pair_similarity_plan numbers it, B, L, Hq, Hkv, S, Tq): remainders of row and key tiles, one and several tiles per split
CASES = [(5, 2, 4, 16, 8, 1300, 1), (6, 2, 3, 16, 4, 900, 12), (2, 9, 3, 8, 8, 1100, 50),
         (7, 1, 3, 8, 2, 700, 70), (1, 24, 2, 16, 4, 261, 20)]


@pytest.mark.parametrize("case", CASES, ids=[f"form{c[0]}" for c in CASES])
@pytest.mark.parametrize("d,dtype", [(72, torch.bfloat16), (80, torch.float16), (96, torch.bfloat16)], ids=["d72", "d80", "d96"])
def test_same_bits_as_padded_heads(case, d, dtype):
    import paper_2507_08045_amd as kr
    form, B, L, Hq, Hkv, S, Tq = case
    gen = torch.Generator(device="cuda").manual_seed(d + form)
    q = torch.randn((B, L, Hq, Tq, d), generator=gen, device="cuda").to(dtype)
    k = torch.randn((B, L, Hkv, S, d), generator=gen, device="cuda").to(dtype)
    padded = [torch.nn.functional.pad(t, (0, 128 - d)).contiguous() for t in (q, k)]
    plans = [kr.plan(kr.make_shape(*t)) for t in ((q, k), padded)]
    assert plans[0]["form"] == form and plans[0] == plans[1]
    for flags in (0, kr.KRUL_FLAG_CAUSAL, kr.KRUL_FLAG_SINGLE_SPLIT):
        got, want = (kr.pair_similarity(*t, scale=0.1, flags=flags, want_head_score=True, want_pair_dist=True) for t in ((q, k), padded))
        torch.cuda.synchronize()
        assert torch.equal(got["head_score"], want["head_score"]) and torch.equal(got["pair_dist"], want["pair_dist"])
    got, want = (kr.pair_similarity_ir(*t, 0.2, scale=0.1) for t in ((q, k), padded))
    torch.cuda.synchronize()
    assert torch.equal(got["ir_mass"], want["ir_mass"])
