"""Plans whose key splits hold several tiles each (running records carried from tile to tile in every split, the last split shorter),
in each tile shape that takes more than 64 rows or 33 to 64, against a float64 evaluation; dense keys, keys in place, the layer test."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu
KEYS = {1: 256, 2: 512, 6: 128, 7: 128}   # per tile of a form (krul_pair_similarity_plan)

# (form, causal, B, L, Hq, Hkv, d, S, Tq)
CASES = [
    (1, False, 5, 3, 16, 8, 64, 2382, 33),
    (1, True, 3, 3, 8, 8, 128, 1835, 135),
    (2, False, 5, 3, 8, 4, 96, 3099, 67),
    (2, True, 3, 3, 2, 2, 64, 10876, 130),
    (6, False, 5, 3, 2, 2, 64, 3100, 133),
    (6, True, 3, 3, 32, 8, 96, 1666, 33),
    (7, False, 5, 3, 4, 4, 128, 3218, 65),
    (7, True, 5, 3, 8, 8, 64, 1581, 72),
]


@pytest.mark.parametrize("form,causal,B,L,Hq,Hkv,d,S,Tq", CASES)
def test_matches_float64(form, causal, B, L, Hq, Hkv, d, S, Tq):
    import paper_2507_08045_amd as kr
    flags = kr.KRUL_FLAG_CAUSAL if causal else 0
    gen = torch.Generator(device="cuda").manual_seed(S)
    q = torch.randn((B, L, Hq, Tq, d), generator=gen, device="cuda").bfloat16()
    k = torch.randn((B, L, Hkv, S, d), generator=gen, device="cuda").bfloat16()
    plan = kr.plan(kr.make_shape(q, k, 0.0, flags))
    assert plan["form"] == form and 1 < plan["n_key_splits"] < -(-S // KEYS[form])
    kd = k.double().repeat_interleave(Hq // Hkv, dim=2).view(B * L * Hq, S, d)
    x = torch.bmm(q.double().view(B * L * Hq, Tq, d), kd.transpose(1, 2).contiguous()).view(B, L, Hq, Tq, S) / math.sqrt(d)
    if causal:
        seen = torch.arange(S, device="cuda")[None, :] <= torch.arange(S - Tq, S, device="cuda")[:, None]
        x = x.masked_fill(~seen, -math.inf)
    w = torch.softmax(x, -1)
    a, b = w[:, :-1], w[:, 1:]
    cos = ((a * b).sum(-1) / torch.sqrt((a * a).sum(-1) * (b * b).sum(-1))).mean(-1)
    dist = torch.sqrt(((a - b) ** 2).sum(-1)).mean((-1, -2))
    # float32 sums over at most 10876 keys, block by block: far below 1e-5 of a cosine or of a distance
    strided = [k[:, l] for l in range(L)]
    for got in (kr.pair_similarity(q, k, flags=flags), kr.pair_similarity_strided(q, strided, flags=flags)):
        torch.cuda.synchronize()
        assert torch.max(torch.abs(got["head_score"] - cos)) <= 1e-5
        assert torch.max(torch.abs(got["pair_dist"] / dist - 1)) <= 1e-5
    if not causal:
        ir = kr.pair_similarity_ir(q, k, 0.2)
        torch.cuda.synchronize()
        mass = torch.cat([w[..., :math.floor(0.1 * S)], w[..., math.floor(0.9 * S):]], -1).sum(-1).mean((-1, -2))
        assert torch.max(torch.abs(ir["ir_mass"] - mass)) <= 1e-5
