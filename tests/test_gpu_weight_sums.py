"""Length of the float32 sums of the weight gradient on the GPU."""
import numpy as np
import pytest
import torch

import dist_inputs as di
from _common import gpu_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "bf16"])
def test_no_float32_sum_runs_over_a_whole_slice(prec):
    """65,536 samples at one point, all with seed s but every 8,192nd with
    2^29 s, which a float32 sum of the terms of s that come after it cannot
    hold: 16 of them are less than half its last place.

    The terms are powers of two times those of one sample alone (bfloat16 and
    float32 keep them exactly), so the exact gradient is (8 2^29 + 65,536 - 8)
    times that sample's.  A sum of at most 1,920 rows (bfloat16; float32: 256)
    loses the terms that follow a large one in it, 1,919 at most; adding such
    sums (up to five to a slice) rounds by at most 32 terms each, and storing
    the total of 2^32 terms by 256.
    """
    from paper_1911_13225_amd import api
    spec = di.C1_SPEC
    Ws, bs = di.make_decoder(spec, seed=5)
    ctx = gpu_ctx(spec, Ws=Ws, bs=bs)
    n, s = 65536, 2.0 ** -9
    p = torch.tensor([[0.21, -0.34, 0.18]], device="cuda")
    z = torch.tensor(di.make_latents(1, spec.latent_dim, sigma=0.1), device="cuda")
    ids = torch.zeros(n, dtype=torch.int32, device="cuda")
    _, w1, b1 = api.dist_sdf_vjp(ctx, p, ids[:1], torch.full((1,), s, device="cuda"), z, prec, want_theta=True)
    sd = torch.full((n,), s, device="cuda")
    sd[::8192] = s * 2.0 ** 29
    _, gW, gb = api.dist_sdf_vjp(ctx, p.expand(n, 3).contiguous(), ids, sd, z, prec, want_theta=True)
    bound = 8 * (1919 + 5 * 32) + 256
    worst = 0.0
    for one, got in zip(w1 + b1, gW + gb):
        one, got = one.double(), got.double()
        k = one != 0
        assert not got[~k].any()
        worst = max(worst, float(((got[k] - (8 * 2.0 ** 29 + n - 8) * one[k]) / one[k]).abs().max()))
    print("terms lost", worst, "of", n, "bound", bound, flush=True)
    assert worst <= bound
    ctx.close()
