"""The gradient through the unrolled march on the GPU: what its bits and its
memory depend on."""
import numpy as np
import pytest
import torch

import dist_inputs as di

pytestmark = pytest.mark.gpu

ENOMEM = -2
# widths of all three padded sizes: column sums in one and in two row groups
MIXED_SPEC = di.DecoderSpec(latent_dim=33, out_dims=(256, 200, 512, 100, 256, 1), skip_layer=2)
NARROW_SPEC = di.DecoderSpec(latent_dim=17, out_dims=(100, 128, 90, 128, 1), skip_layer=2)
SPECS = {"mixed": MIXED_SPEC, "narrow": NARROW_SPEC, "noskip": di.DecoderSpec(20, (128, 256, 1), None)}


def context(spec, budget=0):
    from paper_1911_13225_amd import api
    Ws, bs = di.make_decoder(spec, seed=5)
    return api.Context.from_spec(spec, Ws, bs, hbm_budget=budget)


def tightest(run):
    """run(budget) in the least budget (to 1/2 MiB) that it does not fail in for want of memory."""
    for half in range(1, 400):
        try:
            return half << 19, run(half << 19)
        except Exception as e:
            if getattr(e, "code", ENOMEM) != ENOMEM or "budget" not in str(e):
                raise
    raise AssertionError("no budget is enough")


def gradient(spec, prm, z, cams, pairs, gd, gs, budget):
    from paper_1911_13225_amd import api
    ctx = context(spec, budget)
    try:
        out = api.dist_render_fwd(ctx, cams, z, prm, pairs=pairs, save=True)
        n = len(pairs)
        seeds = gd[:n] * torch.isfinite(out["depth"])
        g = api.dist_render_bwd_unrolled(ctx, out["saved"], seeds, gs[:n], n_latents=z.shape[0])
        assert torch.equal(g, api.dist_render_bwd_unrolled(ctx, out["saved"], seeds, gs[:n], n_latents=z.shape[0]))
        out["saved"].free()
        return g
    finally:
        ctx.close()


# Image sizes whose steps have from under one to 150 tiles: without a cap on the
# memory all steps of a level share chunks, in the least memory the larger steps
# are chunks of their own.
@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "bf16"])
@pytest.mark.parametrize("name,H,W,levels,steps", [("mixed", 28, 36, 2, 50), ("narrow", 96, 100, 0, 12),
                                                   ("noskip", 60, 44, 1, 255), ("mixed", 5, 3, 0, 1)])
def test_unrolled_gradient_bits(name, H, W, levels, steps, prec):
    """An image's gradient is the same, bit for bit, alone and beside others of
    its own and of other latents, with memory for chunks of steps and without."""
    spec = SPECS[name]
    prm = di.TraceParams(max_steps=steps, c2f_levels=levels, precision=prec, want_normals=0, keep_history=1)
    z = torch.tensor(di.make_latents(12, spec.latent_dim, sigma=0.05), device="cuda")
    cams = di.random_sphere_cameras(12, H, W)
    g = torch.Generator(device="cuda").manual_seed(9)
    gd, gs = (torch.randn(12, H, W, generator=g, device="cuda") for _ in range(2))
    # image 0 has latent 5; latents 0, 7 and 11 have no image, latent 3 has two
    pairs = [(0, 5), (1, 1), (2, 9), (3, 3), (4, 2), (5, 4), (6, 3), (7, 6), (8, 10), (9, 8)]
    ref = None
    for n in (1, 2, 10):
        for cap in (False, True):
            run = lambda budget: gradient(spec, prm, z, cams, pairs[:n], gd, gs, budget)
            one = tightest(run)[1] if cap else run(0)
            used = sorted({l for _, l in pairs[:n]})
            assert not one[[l for l in range(12) if l not in used]].any()
            ref = one if ref is None else ref
            assert torch.equal(ref[5], one[5]), (n, cap)
            last = one if not cap else last
            assert torch.equal(last, one), (n, cap)
    assert ref[5].abs().max() > 0


@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "bf16"])
def test_unrolled_gradient_leaves_memory_to_other_calls(prec):
    """In every budget that two renders, their unrolled gradients and a weight
    gradient fit when the gradients come last, they fit when they come first:
    what the first gradient took beyond a step's buffers goes to the others."""
    from paper_1911_13225_amd import api
    spec = di.C1_SPEC
    prm = di.TraceParams(max_steps=50, c2f_levels=2, precision=prec, want_normals=0, keep_history=1)
    z = torch.tensor(di.make_latents(1, spec.latent_dim, sigma=0.05), device="cuda")
    cams = di.random_sphere_cameras(1, 64, 64)
    rng = np.random.Generator(np.random.PCG64(14))
    P = torch.tensor(rng.uniform(-0.6, 0.6, (3000, 3)).astype(np.float32), device="cuda")
    ids = torch.zeros(3000, dtype=torch.int32, device="cuda")
    sd = torch.tensor(rng.standard_normal(3000).astype(np.float32), device="cuda")

    def run(order, budget):
        ctx = context(spec, budget)
        saved, res = {}, {}
        try:
            for what in order:
                if what[0] == "f":
                    out = api.dist_render_fwd(ctx, cams, z, prm, save=True)
                    saved[what[1]] = out["saved"], torch.isfinite(out["depth"]).float()
                elif what[0] == "u":
                    s, fg = saved[what[1]]
                    res[what] = api.dist_render_bwd_unrolled(ctx, s, fg, torch.ones_like(fg), n_latents=1)
                else:
                    res[what] = api.dist_sdf_vjp(ctx, P, ids, sd, z, prec, want_theta=True)[0]
            return res
        finally:
            for s, _ in saved.values():
                s.free()
            ctx.close()

    budget, last = tightest(lambda b: run(("w", "fA", "fB", "uA", "uB"), b))
    print("budget", budget, flush=True)
    for more in range(0, 600 << 20, 8 << 20):
        first = run(("fA", "uA", "fB", "uB", "w"), budget + more)
        for k in last:
            assert torch.equal(first[k], last[k]), (k, more >> 20)


@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "bf16"])
def test_unrolled_gradient_in_a_graph(prec):
    """Captured after one eager call, the gradient replays with new seeds as
    the eager call has it, with eager calls, which take longer chunks, and
    allocations between the replays."""
    from paper_1911_13225_amd import api
    spec = MIXED_SPEC
    prm = di.TraceParams(max_steps=50, c2f_levels=2, precision=prec, want_normals=0, keep_history=1)
    z = torch.tensor(di.make_latents(2, spec.latent_dim, sigma=0.05), device="cuda")
    cams = di.random_sphere_cameras(2, 44, 36)
    ctx = context(spec)
    out = api.dist_render_fwd(ctx, cams, z, prm, save=True)
    n = out["depth"].shape[0]
    fg = torch.isfinite(out["depth"]).float()
    g = torch.Generator(device="cuda").manual_seed(12)
    gd, gs = torch.zeros_like(fg), torch.zeros_like(fg)
    call = lambda: api.dist_render_bwd_unrolled(ctx, out["saved"], gd, gs, n_latents=2)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = call()
    for i in range(4):
        gd.copy_(torch.randn(n, 44, 36, generator=g, device="cuda") * fg)
        gs.copy_(torch.randn(n, 44, 36, generator=g, device="cuda"))
        graph.replay()
        torch.cuda.synchronize()
        one = got.clone()
        assert one.abs().max() > 0 and torch.equal(one, call()), i
        other = api.dist_render_fwd(ctx, cams, z, prm, save=True)
        other["saved"].free()
        torch.cuda.synchronize()
    out["saved"].free()
    ctx.close()


def test_unrolled_gradients_on_two_streams():
    """Calls on two streams share the context's block of memory and wait for
    each other's use of it."""
    from paper_1911_13225_amd import api
    spec = di.C1_SPEC
    prm = di.TraceParams(max_steps=50, c2f_levels=2, precision=1, want_normals=0, keep_history=1)
    z = torch.tensor(di.make_latents(1, spec.latent_dim, sigma=0.05), device="cuda")
    ctx = context(spec)
    handles = []
    for side, seed in ((64, 2000), (96, 3000)):
        out = api.dist_render_fwd(ctx, di.random_sphere_cameras(2, side, side, base_seed=seed), z, prm, save=True)
        handles.append((out["saved"], torch.isfinite(out["depth"]).float()))
    call = lambda i: api.dist_render_bwd_unrolled(ctx, handles[i][0], handles[i][1], torch.ones_like(handles[i][1]),
                                                  n_latents=1)
    ref = [call(0), call(1)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = []
    for _ in range(6):
        for i in (0, 1):
            with torch.cuda.stream(streams[i]):
                got.append((i, call(i)))
    torch.cuda.synchronize()
    for i, g in got:
        assert torch.equal(g, ref[i])
    for s, _ in handles:
        s.free()
    ctx.close()
