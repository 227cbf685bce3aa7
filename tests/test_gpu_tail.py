"""GPU tests of the kernels behind the similarity kernel -- merged records, averages over heads -- at the ends of their ranges."""
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
