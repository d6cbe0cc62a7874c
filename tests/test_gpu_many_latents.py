"""Samples of many latents on the GPU: each latent's gradient as by itself."""
import numpy as np
import pytest
import torch

import dist_inputs as di
from _common import gpu_ctx

pytestmark = pytest.mark.gpu


# Latents from one to more than there are workgroups for their runs of 64 tiles
# (64 x 64 samples), and one latent that owns nearly all samples: several runs
# per workgroup.
@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "bf16"])
@pytest.mark.parametrize("n_lat,heavy", [(1, 20000), (3, 70000), (20000, 70000)])
def test_code_gradient_of_a_latent_among_many(n_lat, heavy, prec):
    """The gradient of the latent with `heavy` samples is the same, bit for bit,
    among n_lat - 1 latents of a few samples each and by itself."""
    from paper_1911_13225_amd import api
    spec = di.C1_SPEC
    Ws, bs = di.make_decoder(spec, seed=5)
    ctx = gpu_ctx(spec, Ws=Ws, bs=bs)
    rng = np.random.Generator(np.random.PCG64(13))
    own = n_lat // 2
    ids = np.concatenate([np.full(heavy, own), rng.integers(0, n_lat, 500)]).astype(np.int32)
    keep = np.nonzero(ids == own)[0]
    P = torch.tensor(rng.uniform(-0.6, 0.6, (ids.size, 3)).astype(np.float32), device="cuda")
    sd = torch.tensor(rng.standard_normal(ids.size).astype(np.float32), device="cuda")
    z = torch.tensor(rng.standard_normal((n_lat, spec.latent_dim)).astype(np.float32) * 0.05, device="cuda")
    t = torch.tensor(ids, device="cuda")
    k = torch.tensor(keep, device="cuda")
    g = api.dist_sdf_vjp(ctx, P, t, sd, z, prec)
    one = api.dist_sdf_vjp(ctx, P[k].contiguous(), torch.zeros(keep.size, dtype=torch.int32, device="cuda"),
                           sd[k].contiguous(), z[own:own + 1].contiguous(), prec)
    assert torch.equal(g[own], one[0])
    empty = torch.ones(n_lat, dtype=torch.bool, device="cuda")
    empty[t.unique().long()] = False
    assert not g[empty].any()
    # a latent of few samples, likewise
    l = int(ids[-1])
    k = torch.tensor(np.nonzero(ids == l)[0], device="cuda")
    one = api.dist_sdf_vjp(ctx, P[k].contiguous(), torch.zeros(k.numel(), dtype=torch.int32, device="cuda"),
                           sd[k].contiguous(), z[l:l + 1].contiguous(), prec)
    assert torch.equal(g[l], one[0])
    ctx.close()
