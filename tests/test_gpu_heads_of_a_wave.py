"""Few query tokens: a wave takes several heads of a kv head.  Groups of heads and tokens that fill its lanes, leave some over or need several waves, with
few and many key splits, written and added to running sums."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_util
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return gpu_util


# heads per kv head, tokens, keys
CASES = [(1, 1, 40), (3, 1, 700), (4, 1, 9000), (5, 3, 300), (8, 8, 700), (16, 5, 130), (70, 1, 64), (24, 7, 2600)]


@pytest.mark.parametrize("case", CASES, ids=[f"{g}heads-{t}tokens-{s}keys" for g, t, s in CASES])
def test_scores_and_running_sums(G, oracle, case):
    import paper_2507_08045_amd as kr
    g, Tq, S = case
    w = workloads.make("heads-of-a-wave", B=2, L=3, Hq=2 * g, Hkv=2, d=64, S=S, Tq=Tq, dtype="bf16", seed=7 + g)
    want = oracle.pair_similarity(w.q, w.k)
    q, k = G.to_device(w)
    out = kr.pair_similarity(q, k, want_head_score=True, want_pair_dist=True)
    start = torch.arange(2 * 2 * 2 * g, dtype=torch.float32, device="cuda").view(2, 2, 2 * g)   # (whole numbers: exact)
    head_sum, dist_sum = start.clone(), start.clone()
    kr.pair_similarity_accumulate(q, k, head_sum, dist_sum)
    torch.cuda.synchronize()
    head, dist = out["head_score"].cpu().numpy(), out["pair_dist"].cpu().numpy()
    # an exponential is known to 7e-7 (logits below 16 to 2^-20); a cosine or a distance of one row of tens of keys moves by about as much
    e = [np.max(np.abs(head - want["head_score"])), np.max(np.abs(dist - want["pair_dist"]))]
    print(f"[{g} heads, {Tq} tokens, {S} keys] cos {e[0]:.1e} dist {e[1]:.1e}", flush=True)
    assert max(e) <= 2e-6
    # sums of up to 560 are rounded to 2^-15
    assert np.max(np.abs((head_sum - start).cpu().numpy() - Tq * head)) <= 2.0 ** -14 + Tq * 1e-6
    assert np.max(np.abs((dist_sum - start).cpu().numpy().mean(-1) - Tq * dist)) <= 2.0 ** -14 + Tq * 1e-6
