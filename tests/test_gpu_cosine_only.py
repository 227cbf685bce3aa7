"""Calls that do not ask for the distance, against the oracle: every tile shape of the 16-bit kernels, heads on four, six and eight MFMAs a
block, both types, keys dense, with strides and in pages, with and without the causal mask.  The keys at the edges of tiles are twice
as long as the others, so that their weights are large and none can be lost or counted twice unseen.  And the same scores where the
distance is asked for."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# form as krul_pair_similarity_plan numbers it, B, L, Hq, Hkv, S, Tq, whether the form is that of the causal call
CASES = [(5, 2, 4, 16, 8, 1300, 1, False), (6, 2, 3, 16, 4, 900, 12, False), (2, 9, 3, 8, 8, 1100, 50, False),
         (7, 1, 3, 8, 2, 700, 70, True), (1, 24, 2, 16, 4, 261, 20, False)]
HEADS = [(64, torch.bfloat16), (64, torch.float16), (40, torch.float16), (96, torch.bfloat16), (72, torch.float16),
         (128, torch.bfloat16), (128, torch.float16)]
DEEP = [((4, 24, 2, 2, 2, 2488, 1, False), 64, torch.bfloat16), ((4, 24, 2, 2, 2, 2488, 1, False), 128, torch.float16),
        ((10, 2, 4, 16, 4, 12001, 121, False), 64, torch.bfloat16), ((10, 2, 4, 16, 4, 12001, 128, False), 40, torch.float16),
        ((10, 3, 6, 16, 4, 4999, 300, False), 64, torch.float16)]
ALL = [(c, d, t) for c in CASES for d, t in HEADS] + DEEP

# A logit is known to 2^-20 (float32 below 16), an exponential to 7e-7 of itself, and a mean of cosines of rows of hundreds of keys to a fraction
# of that: at most 1.8e-7 in the cases below.  (With one key at a tile's edge lost: 2.6e-6 for one row of 2488 keys,
# 1e-3 mostly.)
TOL = 1e-6


def keys_in_place(k):
    """The keys in a [B][S][Hkv][d] cache per layer, and in pages of 16 whose unused slots hold NaN."""
    import paper_2507_08045_amd as kr
    B, L, Hkv, S, d = k.shape
    pages = -(-S // 16)
    table = torch.randperm(B * pages, generator=torch.Generator().manual_seed(S)).int().cuda().view(B, pages)
    pools = []
    for l in range(L):
        tokens = torch.nn.functional.pad(k[:, l].transpose(1, 2), (0, 0, 0, 0, 0, pages * 16 - S), value=float("nan"))
        pool = torch.empty((B * pages, 16, Hkv, d), dtype=k.dtype, device="cuda")
        pool[table.long()] = tokens.reshape(B, pages, 16, Hkv, d)
        pools.append(pool)
    return {"strided": kr.StridedKeys([k[:, l].transpose(1, 2).contiguous().transpose(1, 2) for l in range(L)]),
            "paged": kr.PagedKeys(pools, table, S)}


@pytest.mark.parametrize("case,d,dtype", ALL, ids=[f"form{c[0]}-{c[5]}keys-d{d}-{str(t)[6:]}" for c, d, t in ALL])
def test_matches_oracle_on_every_source_of_keys(oracle, case, d, dtype):
    import paper_2507_08045_amd as kr
    form, B, L, Hq, Hkv, S, Tq, causal = case
    gen = torch.Generator(device="cuda").manual_seed(S + d)
    q = torch.randn((B, L, Hq, Tq, d), generator=gen, device="cuda")
    q[:, 1:] = 0.6 * q[:, 1:] + 0.8 * q[:, :1]   # (layers that are alike, as a model's are)
    k = torch.randn((B, L, Hkv, S, d), generator=gen, device="cuda")
    k[:, 1:] = 0.6 * k[:, 1:] + 0.8 * k[:, :1]
    at = torch.arange(S, device="cuda")
    k[..., (at % 128 == 0) | (at % 128 == 127) | (at == S - 1), :] *= 2
    q, k = q.to(dtype), k.to(dtype)
    host = [(t.view(torch.int16).cpu().numpy().view(np.uint16) if dtype == torch.bfloat16 else t.cpu().numpy()) for t in (q, k)]
    units = sorted({(0, 0, 0), (B - 1, L - 2, Hq - 1), (B // 2, 0, Hq // 2), (B - 1, (L - 1) // 2, 1), (0, L - 2, Hq // 3)})
    places = tuple(np.array(units).T)
    assert kr.plan(kr.make_shape(q, k, 0.0, kr.KRUL_FLAG_CAUSAL if causal else 0))["form"] == form
    sources = keys_in_place(k)
    for flags in (0, kr.KRUL_FLAG_CAUSAL):
        want, _ = oracle.unit_scores(*host, units, causal=bool(flags))
        got = kr.pair_similarity(q, k, flags=flags, want_head_score=True, want_pair_dist=False)
        sums = {"dense": torch.zeros((B, L - 1, Hq), device="cuda")}
        kr.pair_similarity_accumulate(q, k, sums["dense"], flags=flags)
        for name, keys in sources.items():
            sums[name] = torch.zeros((B, L - 1, Hq), device="cuda")
            kr.pair_similarity_accumulate_in_place(q, keys, sums[name], flags=flags)
        both = kr.pair_similarity(q, k, flags=flags, want_head_score=True, want_pair_dist=True)
        torch.cuda.synchronize()
        assert torch.equal(got["head_score"], both["head_score"]) and torch.equal(got["pair_score"], both["pair_score"])
        for name, head in {"mean": got["head_score"], **{n: s / Tq for n, s in sums.items()}}.items():
            err = np.max(np.abs(head.cpu().numpy()[places] - want))
            print(f"[{form} d{d} {dtype} flags {flags} {name}] {err:.2e}", flush=True)
            assert err <= TOL, (name, flags, err)
