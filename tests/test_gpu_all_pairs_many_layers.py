"""GPU parity of the all-pairs kernels that keep the exponentials in memory, which every model of more than 32 layers takes: keys
in place, causal rows, binary16, head sizes between 64 and 128 and below, several conversations, row groups of one, two, four and eight
32-row blocks, batches that cut a conversation's rows."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

# (name, B, L, Hq, Hkv, d, S, Tq, dtype, causal)
CASES = [
    ("33-layers-d96", 1, 33, 6, 2, 96, 300, 20, "f16", False),
    ("36-layers-d80-groups-of-four", 2, 36, 5, 1, 80, 200, 22, "bf16", False),
    ("40-layers-causal-groups-of-eight", 1, 40, 4, 1, 128, 260, 60, "bf16", True),
    ("64-layers-d40", 1, 64, 4, 2, 40, 161, 17, "bf16", False),
    ("65-layers-causal", 1, 65, 4, 1, 64, 140, 33, "f16", True),
    ("80-layers-two-row-groups", 1, 80, 5, 1, 128, 129, 53, "bf16", False),
    ("97-layers-d72", 2, 97, 2, 1, 72, 97, 5, "f16", False),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_matches_oracle(oracle, case):
    import gpu_util as G
    import paper_2507_08045_amd as kr
    name, B, L, Hq, Hkv, d, S, Tq, dtype, causal = case
    rng = np.random.default_rng(L * S)
    w = workloads.make(name, B=B, L=L, Hq=Hq, Hkv=Hkv, d=d, S=S, Tq=Tq, dtype=dtype, rho_k=rng.uniform(0.5, 0.95, size=(B, L - 1, Hkv)), seed=62)
    q, k = G.to_device(w)
    flags = kr.KRUL_FLAG_CAUSAL if causal else 0
    want, tol = oracle.all_pairs(w.q, w.k, causal=causal), G.all_pairs_tolerance(q, k, causal, split=128)
    # keys in one cache per layer, and in 16-key pages (their unused slots hold NaN)
    strided = kr.StridedKeys([k[:, l].permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for l in range(L)])
    blocks = -(-S // 16)
    table = torch.from_numpy(rng.permutation(B * blocks)).cuda().view(B, blocks)
    pools = []
    for l in range(L):
        tokens = torch.full((B, blocks * 16, Hkv, d), float("nan"), dtype=k.dtype, device="cuda")
        tokens[:, :S] = k[:, l].permute(0, 2, 1, 3)
        pool = torch.empty((B * blocks, 16, Hkv, d), dtype=k.dtype, device="cuda")
        pool[table.view(-1)] = tokens.view(B * blocks, 16, Hkv, d)
        pools.append(pool)
    paged = kr.PagedKeys(pools, table.to(torch.int32).contiguous(), S)
    for source, keys in (("dense", k), ("strided", strided), ("paged", paged)):
        out = kr.all_pairs_similarity_in_place(q, keys, want_head_score=True, flags=flags)
        torch.cuda.synchronize()
        G.assert_all_pairs(out, want, tol, f"{name} {source}")
    # the smallest workspace: a row group at a time, the same bits
    small = torch.empty(kr.all_pairs_workspace_bytes(kr.make_shape(q, k, 0.0, flags), 1), dtype=torch.uint8, device="cuda")
    full = kr.all_pairs_similarity(q, k, want_head_score=True, flags=flags)
    cut = kr.all_pairs_similarity(q, k, want_head_score=True, flags=flags, workspace=small)
    torch.cuda.synchronize()
    for n in ("head_score", "pair_score", "pair_dist"):
        assert torch.equal(full[n], cut[n]), f"{name} {n}"
