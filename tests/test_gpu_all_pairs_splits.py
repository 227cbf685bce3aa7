"""GPU parity of the all-pairs kernel that keeps the exponentials in LDS where its key splits fill one to several rounds of
workgroups, with numbers of row blocks that divide neither 8 nor 256 -- in one batch and in the smallest batches, which must give the
same bits."""
import ctypes

import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

# (name, B, L, Hq, Hkv, d, S, Tq): row blocks of the problem -> splits
CASES = [
    ("72-blocks", 1, 5, 32, 8, 64, 700, 72),
    ("27-blocks-one-row-over", 1, 9, 9, 3, 72, 1030, 86),
    ("288-blocks", 3, 3, 32, 8, 64, 260, 90),
    ("one-block", 1, 4, 2, 1, 128, 4200, 3),   # 128 splits, the most
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_matches_oracle_whatever_the_batch(oracle, case):
    import gpu_util as G
    import paper_2507_08045_amd as kr
    name, B, L, Hq, Hkv, d, S, Tq = case
    w = workloads.make(name, B=B, L=L, Hq=Hq, Hkv=Hkv, d=d, S=S, Tq=Tq, dtype="bf16",
                       rho_k=np.random.default_rng(S).uniform(0.5, 0.95, size=(B, L - 1, Hkv)), seed=73)
    q, k = G.to_device(w)
    out = kr.all_pairs_similarity(q, k, want_head_score=True)
    torch.cuda.synchronize()
    G.assert_all_pairs(out, oracle.all_pairs(w.q, w.k), G.all_pairs_tolerance(q, k, False), name)
    least = kr.binding.lib().krul_all_pairs_workspace(ctypes.byref(kr.make_shape(q, k)), 1)
    small = kr.all_pairs_similarity(q, k, want_head_score=True, workspace=torch.empty(least, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    for n in ("pair_score", "pair_dist", "head_score"):
        assert torch.equal(out[n], small[n])
