"""Device memory on the GPU: calls that get none, and calls that run after them."""
import numpy as np
import pytest
import torch

import dist_inputs as di
from _common import gpu_ctx

pytestmark = pytest.mark.gpu


def test_a_failed_allocation_ends_with_its_own_call():
    """A call that the device has no memory for reports it; the next call of
    the same thread runs and reports its own outcome."""
    from paper_1911_13225_amd import api, _native as N
    spec = di.C1_SPEC
    Ws, bs = di.make_decoder(spec, seed=5)
    ctx = gpu_ctx(spec, Ws=Ws, bs=bs)
    P = torch.tensor(np.random.default_rng(3).uniform(-0.7, 0.7, (100, 3)).astype(np.float32), device="cuda")
    ids = torch.zeros(100, dtype=torch.int32, device="cuda")
    z = torch.tensor(di.make_latents(1, spec.latent_dim, sigma=0.1), device="cuda")
    ref = api.dist_sdf_eval(ctx, P, ids, z, 0)
    # the folded biases of n_lat codes take 4 KB each, more than twice the
    # device's memory: the call ends at their allocation, before any launch
    n_lat = torch.cuda.get_device_properties(0).total_memory // 2048
    f = torch.empty_like(ref)
    p = api._ptr
    rc = N.load().dist_sdf_eval(ctx.handle, p(P), p(ids), p(z), n_lat, 100, 0, p(f), api._stream())
    assert rc in (-2, -6), rc                       # DIST_ENOMEM, DIST_EHIP
    assert torch.equal(api.dist_sdf_eval(ctx, P, ids, z, 0), ref)
    assert torch.equal(torch.ones(3, device="cuda") + 1, torch.full((3,), 2.0, device="cuda"))
    ctx.close()
