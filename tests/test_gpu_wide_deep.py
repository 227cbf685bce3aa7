"""Long calls of models with heads of up to 64 elements run in tiles of 128 x 512: the scores of the same inputs with zeros added up to 72 elements, which take
other tiles, on dense keys, keys with strides and keys in pages, with and without the causal mask."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# (B, L, Hq, Hkv, d, S, Tq): several tiles a split with remainders of rows and keys, a head below 64, whole tiles
CASES = [(2, 24, 16, 4, 64, 12001, 121), (2, 24, 16, 4, 40, 12001, 128), (1, 24, 16, 4, 64, 4096, 512)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"d{c[4]}-{c[6]}-over-{c[5]}")
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16], ids=["bf16", "f16"])
def test_matches_other_tiles(case, dtype):
    import paper_2507_08045_amd as kr
    B, L, Hq, Hkv, d, S, Tq = case
    gen = torch.Generator(device="cuda").manual_seed(S)
    q = torch.randn((B, L, Hq, Tq, d), generator=gen, device="cuda").to(dtype)
    k = torch.randn((B, L, Hkv, S, d), generator=gen, device="cuda").to(dtype)
    padded = [torch.nn.functional.pad(t, (0, 72 - d)).contiguous() for t in (q, k)]
    pages = -(-S // 16)
    table = torch.randperm(B * pages, generator=torch.Generator().manual_seed(1)).int().cuda().view(B, pages)
    pools = []
    for l in range(L):
        pool = torch.zeros((B * pages, 16, Hkv, d), dtype=dtype, device="cuda")
        tokens = torch.nn.functional.pad(k[:, l].transpose(1, 2), (0, 0, 0, 0, 0, pages * 16 - S))
        pool[table.long()] = tokens.reshape(B, pages, 16, Hkv, d)
        pools.append(pool)
    in_place = [kr.StridedKeys([k[:, l].transpose(1, 2).contiguous().transpose(1, 2) for l in range(L)]), kr.PagedKeys(pools, table, S)]
    for flags in (0, kr.KRUL_FLAG_CAUSAL):
        assert kr.plan(kr.make_shape(q, k, 0.125, flags))["form"] == 10
        assert kr.plan(kr.make_shape(*padded, 0.125, flags))["form"] != 10
        got, want = (kr.pair_similarity(*t, scale=0.125, flags=flags) for t in ((q, k), padded))
        # the logits are the same bits and the sums of float32 are in another order: terms that round at random (7e-8 is seen), means of thousands
        assert torch.max(torch.abs(got["head_score"] - want["head_score"])) <= 1e-6
        assert torch.max(torch.abs(got["pair_dist"] - want["pair_dist"])) <= 1e-6
        for keys in in_place:
            cos, dist = (torch.zeros((B, L - 1, Hq), device="cuda") for _ in range(2))
            kr.pair_similarity_accumulate_in_place(q, keys, cos, dist, scale=0.125, flags=flags)
            # (and a sum of Tq of them, rounded to 2^-24 of itself in each of its dozen joins, divided by Tq)
            assert torch.max(torch.abs(cos / Tq - want["head_score"])) <= 2e-6
            assert torch.max(torch.abs((dist / Tq).mean(-1) - want["pair_dist"])) <= 2e-6
