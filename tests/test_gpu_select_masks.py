"""The greedy choice by masks at the ends of its words: layers around 64 and 128, rising, falling, equal and missing scores, against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

KINDS = {
    "rising": lambda rng, n: np.arange(n, dtype=np.float32),
    "falling": lambda rng, n: -np.arange(n, dtype=np.float32),
    "equal": lambda rng, n: np.zeros(n, np.float32) * rng.choice([1.0, -1.0], n).astype(np.float32),   # 0 and -0
    "ties": lambda rng, n: rng.integers(0, 3, n).astype(np.float32),
    "ends": lambda rng, n: rng.choice(np.array([np.inf, -np.inf, np.nan, 1.0, 1e-45], np.float32), n),
}


@pytest.mark.parametrize("layers", [2, 3, 63, 64, 65, 66, 127, 128, 129])
def test_against_the_oracle(oracle, layers):
    import paper_2507_08045_amd as kr
    rng = np.random.default_rng(layers)
    scores = np.stack([f(rng, layers - 1) for f in KINDS.values()])
    eligible = rng.random((len(KINDS), layers)) < 0.8
    eligible[0] = True
    for n_select in {0, 1, layers // 4, layers // 2}:
        for el in (None, eligible.astype(np.uint8)):
            pairs, count = kr.select_pairs(torch.from_numpy(scores).cuda(), n_select, None if el is None else torch.from_numpy(el).cuda())
            torch.cuda.synchronize()
            want_pairs, want_count = oracle.select_pairs(scores.astype(np.float64), n_select, el)
            np.testing.assert_array_equal(pairs.cpu().numpy(), want_pairs, err_msg=f"{list(KINDS)} n_select={n_select}")
            np.testing.assert_array_equal(count.cpu().numpy(), want_count)
