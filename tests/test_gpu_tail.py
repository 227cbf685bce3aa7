"""GPU tests of the kernels behind the similarity kernel -- merged records, averages over heads -- at the ends of their ranges."""
import ctypes
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
def test_mass_far_below_the_largest_exponential(dtype):
    """The first and last keys' logits lie 129.8 powers of two below the others', in key splits of their own: the mass on T_initial and
    T_recent is a subnormal number, not zero."""
    import paper_2507_08045_amd as kr
    S = 1024
    q = torch.zeros((1, 2, 1, 1, 64), dtype=dtype, device="cuda")
    q[..., 0] = 1.0
    k = torch.zeros((1, 2, 1, S, 64), dtype=dtype, device="cuda")
    k[:, :, :, 256:768, 0] = 90.0
    assert kr.plan(kr.make_shape(q, k, 1.0))["n_key_splits"] >= 4
    out = kr.pair_similarity_ir(q, k, 1e-41, scale=1.0)
    torch.cuda.synchronize()
    want = (102 + 103) / 512 * 2.0 ** (-90 * math.log2(math.e))       # keys [0, 102) and [921, 1024); e^-90
    got = out["ir_mass"].cpu().double()
    # 2^-149 is 5e-6 of it, and the exponent of a float32 near 130 is known to 2^-17: 1e-4 covers both
    assert torch.all(torch.abs(got / want - 1) <= 1e-4), (got, want)
    assert out["eligible"].cpu().tolist() == [[1, 1]]


def test_more_pairs_than_one_launch_numbers():
    """2^27 pairs and a few: 32 threads for each are more than the 2^32 that a launch can number."""
    import paper_2507_08045_amd as kr
    batch, pairs = 2 ** 25 + 1, 4
    sums = torch.arange(batch * pairs, dtype=torch.int32, device="cuda").remainder_(8191).float().view(batch, pairs, 1)
    out = kr.pair_scores_from_sums(sums, 2.0)
    torch.cuda.synchronize()
    assert torch.equal(out["pair_score"], sums.view(batch, pairs) * 0.5)   # (one head, a power of two: exact)


def test_more_heads_than_one_launch_numbers():
    """Scores and the layer test in one launch: 3 * 5.9 million (layer or pair, head) values are more than 2^24 workgroups."""
    import paper_2507_08045_amd as kr
    B, Hq, S, Tq, d = 92001, 64, 4, 9, 8
    gen = torch.Generator(device="cuda").manual_seed(5)
    q = torch.randn((B, 2, Hq, Tq, d), generator=gen, device="cuda").bfloat16()
    k = torch.randn((B, 2, 1, S, d), generator=gen, device="cuda").bfloat16()
    out = kr.pair_similarity_ir(q, k, 0.5)
    torch.cuda.synchronize()
    x = torch.matmul(q.float().view(B, 2, Hq * Tq, d), k.float().view(B, 2, S, d).transpose(-1, -2).contiguous()) / math.sqrt(d)
    p = torch.softmax(x, -1).view(B, 2, Hq, Tq, S)
    a, r = p[:, 0], p[:, 1]
    cos = ((a * r).sum(-1) / torch.sqrt((a * a).sum(-1) * (r * r).sum(-1))).mean(-1)
    mass = p[..., 3].mean((-1, -2))   # T_recent of four keys; T_initial is empty
    # float32 on both sides, sums of 4 keys and 9 rows
    assert torch.max(torch.abs(out["head_score"][:, 0] - cos)) <= 1e-5
    assert torch.max(torch.abs(out["ir_mass"] - mass)) <= 1e-5


def test_head_scores_in_the_place_of_their_sums():
    """krul_pair_scores_from_sums with head_score = head_sum: every sum is read once, before its scaled value takes its place."""
    import paper_2507_08045_amd as kr
    B, NP, Hq = 3, 5, 70
    sums = torch.rand((B, NP, Hq), generator=torch.Generator().manual_seed(1)).cuda() * 7.0
    want = kr.pair_scores_from_sums(sums, 7.0)
    vp, pair = ctypes.c_void_p, torch.empty((B, NP), device="cuda")
    rc = kr.lib().krul_pair_scores_from_sums(vp(sums.data_ptr()), None, B, NP + 1, Hq, 7.0, vp(pair.data_ptr()), vp(sums.data_ptr()), None,
                                             vp(torch.cuda.current_stream().cuda_stream))
    assert rc == kr.KRUL_OK
    torch.cuda.synchronize()
    assert torch.equal(pair, want["pair_score"]) and torch.equal(sums, want["head_score"])
