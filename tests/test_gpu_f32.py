"""GPU parity of the float32 kernel (operands split into three bfloat16 planes) at float32 accuracy: head sizes around
its steps, row counts around its tiles, key splits of one and of several tiles, causal splits without a key, keys in
pages; and 16-bit inputs with heads above 128, which take the same kernel."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
TOL32 = 5e-6   # cosines and distances of float32 logits (sums of 8..256 products, softmax sums of up to 2000 keys)

# (name, B, L, Hq, Hkv, d, S, Tq, dtype)
CASES = [
    ("d8", 1, 3, 2, 1, 8, 130, 5, "f32"),
    ("d64-rows31", 1, 4, 1, 1, 64, 127, 31, "f32"),
    ("d72-rows33", 1, 3, 3, 1, 72, 129, 11, "f32"),
    ("d96-rows65", 2, 3, 5, 1, 96, 257, 13, "f32"),
    ("d104-rows64", 1, 3, 4, 2, 104, 300, 32, "f32"),
    ("d128-one-key", 1, 5, 4, 2, 128, 1, 1, "f32"),
    ("d128-rows200", 1, 9, 8, 2, 128, 1500, 50, "f32"),
    ("d136", 1, 3, 4, 2, 136, 520, 9, "f32"),
    ("d256", 1, 3, 4, 2, 256, 300, 7, "f32"),
    # three row blocks on eight waves, 256-key tiles: the least rows and the most of one tile, two tiles, keys of one tile, a ragged second one
    ("three-blocks-rows65", 8, 17, 32, 32, 96, 200, 65, "f32"),
    ("three-blocks-rows80", 16, 16, 16, 4, 128, 511, 20, "f32"),
    ("three-blocks-rows96", 1, 32, 32, 8, 128, 1021, 24, "f32"),
    ("three-blocks-rows186", 1, 9, 32, 32, 128, 300, 186, "f32"),
    ("bf16-d136", 1, 4, 4, 2, 136, 300, 20, "bf16"),
    ("f16-d256", 1, 3, 4, 2, 256, 200, 40, "f16"),
]


def rows_per_tile(q, k, flags):
    import paper_2507_08045_amd as kr
    return kr.plan(kr.make_shape(q, k, flags=flags))["rows_per_tile"]


def in_pages(k):
    """The keys [B, L, Hkv, S, d] in pages of 16 tokens: pools of the layers, block table."""
    B, L, Hkv, S, d = k.shape
    blocks = -(-S // 16)
    table = torch.randperm(B * blocks, device="cuda").view(B, blocks)
    pools = []
    for l in range(L):
        pool = torch.zeros((B * blocks, 16, Hkv, d), dtype=k.dtype, device="cuda")
        padded = torch.zeros((B, blocks * 16, Hkv, d), dtype=k.dtype, device="cuda")
        padded[:, :S] = k[:, l].permute(0, 2, 1, 3)
        pool[table.view(-1)] = padded.view(B * blocks, 16, Hkv, d)
        pools.append(pool)
    return pools, table.to(torch.int32)


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_f32_kernel_matches_oracle(oracle, case):
    import gpu_util as G
    import paper_2507_08045_amd as kr
    name, B, L, Hq, Hkv, d, S, Tq, dtype = case
    w = workloads.make(name, B=B, L=L, Hq=Hq, Hkv=Hkv, d=d, S=S, Tq=Tq, dtype=dtype, seed=411,
                       rho_k=np.random.default_rng(6).uniform(0.4, 0.95, size=(B, L - 1, Hkv)))
    q, k = G.to_device(w)
    if name.startswith("three-blocks"):
        assert rows_per_tile(q, k, 0) == 96
    want = oracle.pair_similarity(w.q, w.k)
    for flags in (0, kr.KRUL_FLAG_SINGLE_SPLIT):   # the second: one workgroup along the keys walks all tiles
        got = G.gpu_scores(q, k, flags=flags)
        for n in ("head_score", "pair_score", "pair_dist"):
            G.assert_close(got[n], want[n], TOL32, f"{name} {n} flags={flags}")
    ir = kr.pair_similarity_ir(q, k, 0.2)
    torch.cuda.synchronize()
    G.assert_close(ir["ir_mass"].cpu().numpy(), oracle.ir_mass(w.q, w.k, 0.2)[0], TOL32, f"{name} ir_mass")
    if S >= Tq:
        gc, wc = G.gpu_scores(q, k, flags=kr.KRUL_FLAG_CAUSAL), oracle.pair_similarity(w.q, w.k, causal=True)
        G.assert_close(gc["head_score"], wc["head_score"], TOL32, f"{name} causal head_score")
    # keys in pages give the dense call's bits
    paged = kr.pair_similarity_paged(q, *in_pages(k), S)
    dense = kr.pair_similarity(q, k)
    torch.cuda.synchronize()
    assert torch.equal(paged["head_score"], dense["head_score"]), name


# (name, B, L, Hq, Hkv, d, S, Tq, all keys in one split, keys of a split, pieces of the layers): 96-row tiles, heads that fill the steps of 16 elements
# or not, splits of several tiles, whose running records (the layer test's too) then come from memory or, of another piece's layer, from LDS
THREE_BLOCKS = [
    ("d72", 1, 33, 16, 16, 72, 511, 65, True, 512, 16),
    ("d88-rows-end-in-both-tiles", 2, 5, 24, 24, 88, 390, 186, True, 512, 2),
    ("d96-chain", 8, 3, 24, 24, 96, 511, 65, True, 512, 1),
    ("d104", 1, 33, 16, 16, 104, 511, 65, True, 512, 16),
    ("d120-rows-end-in-both-tiles", 2, 5, 24, 24, 120, 390, 186, True, 512, 2),
    ("d120-one-tile", 1, 17, 32, 32, 120, 300, 65, False, 256, 4),
    ("d128-two-splits", 4, 3, 24, 24, 128, 1000, 65, False, 512, 1),
    ("d128-grouped", 1, 32, 32, 8, 128, 3000, 24, False, 768, 8),
]


@pytest.mark.parametrize("case", THREE_BLOCKS, ids=[c[0] for c in THREE_BLOCKS])
def test_three_row_blocks(oracle, case):
    import gpu_util as G
    import paper_2507_08045_amd as kr
    name, B, L, Hq, Hkv, d, S, Tq, single, keys_per_split, pieces = case
    flags = kr.KRUL_FLAG_SINGLE_SPLIT if single else 0
    w = workloads.make(name, B=B, L=L, Hq=Hq, Hkv=Hkv, d=d, S=S, Tq=Tq, dtype="f32", seed=413,
                       rho_k=np.random.default_rng(7).uniform(0.4, 0.95, size=(B, L - 1, Hkv)))
    q, k = G.to_device(w)
    for f in (flags, flags | kr.KRUL_FLAG_CAUSAL):
        plan = kr.plan(kr.make_shape(q, k, flags=f))
        assert (plan["rows_per_tile"], plan["keys_per_split"], plan["n_layer_chunks"]) == (96, keys_per_split, pieces), plan
    got, want = G.gpu_scores(q, k, flags=flags), oracle.pair_similarity(w.q, w.k)
    for n in ("head_score", "pair_score", "pair_dist"):
        G.assert_close(got[n], want[n], TOL32, f"{name} {n}")
    ir = kr.pair_similarity_ir(q, k, 0.2, flags=flags)
    paged = kr.pair_similarity_paged(q, *in_pages(k), S, flags=flags)
    torch.cuda.synchronize()
    G.assert_close(ir["ir_mass"].cpu().numpy(), oracle.ir_mass(w.q, w.k, 0.2)[0], TOL32, f"{name} ir_mass")
    np.testing.assert_array_equal(paged["head_score"].cpu().numpy(), got["head_score"])
    gc, wc = G.gpu_scores(q, k, flags=flags | kr.KRUL_FLAG_CAUSAL), oracle.pair_similarity(w.q, w.k, causal=True)
    for n in ("head_score", "pair_dist"):
        G.assert_close(gc[n], wc[n], TOL32, f"{name} causal {n}")


def test_causal_whole_prompt_f32(oracle):
    import gpu_util as G
    import paper_2507_08045_amd as kr
    w = workloads.make("f32-causal", B=1, L=5, Hq=2, Hkv=1, d=64, S=700, Tq=700, dtype="f32", seed=412, rho_k=0.8)
    q, k = G.to_device(w)
    got, want = G.gpu_scores(q, k, flags=kr.KRUL_FLAG_CAUSAL), oracle.pair_similarity(w.q, w.k, causal=True)
    G.assert_close(got["head_score"], want["head_score"], TOL32, "causal head_score")


def test_logits_are_not_biased():
    """Elements whose third plane would always have the operand's sign if the planes were cut off instead of rounded: every product
    then misses 2^-21 of itself, and the logit of eight of them four units of its last place.  Rounding alone -- the small terms' sum, its
    addition to the large one's, the scaling, half a unit each at most -- can move the difference of the two logits by less than half of that."""
    import math
    import paper_2507_08045_amd as kr
    x = 1.0 + 2.0 ** -7 - 2.0 ** -23
    scale = 2.0 ** 17
    q = torch.full((1, 2, 1, 1, 8), x, device="cuda")
    k = torch.ones((1, 2, 1, 2, 8), device="cuda")
    k[0, 0, 0, 0] = x                                     # layer 0, key 0: eight products x * x
    k[0, 0, 0, 1, :4] = 1.0 + 2.0 ** -6                   # key 1: a sum close to it of products without a third plane
    k[0, 1, 0, 1] = -1.0                                  # layer 1: all weight on key 0
    out = kr.pair_similarity(q, k, scale=scale)
    torch.cuda.synchronize()
    cos = out["pair_score"].item()                        # of (p0, 1 - p0) and (1, 0)
    log2_ratio = math.log2(cos / math.sqrt(1.0 - cos * cos))
    c = scale * math.log2(math.e)
    want = c * 8 * x * (x - 1.0 - 2.0 ** -7)
    ulp = 2.0 ** -20                                      # of a logit between 8 and 16
    rounding = 2 * c * ulp * 0.5 + 2 * 0.5 * 2.0 ** -3    # (two logits: the addition, and the scaled value between 2^20 and 2^21)
    assert abs(log2_ratio - want) <= rounding + 1e-3, (log2_ratio, want, rounding)
