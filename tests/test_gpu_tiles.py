"""Tile heights of the decoder kernels on the GPU.

A launch takes its rows in tiles of 128, 64, 32 or 16 rows, chosen by their
number.  A row's value does not depend on the tile that holds it, so every
count around a tile's edge is checked against the same rows of one large
launch, bit for bit, and against the FP64 oracle.
"""
import numpy as np
import pytest
import torch

import dist_inputs as di
from _common import gpu_ctx, oracle_decoder

pytestmark = pytest.mark.gpu

# widths of all three padded sizes, two of them between layers and at the skip
MIXED_SPEC = di.DecoderSpec(latent_dim=33, out_dims=(256, 200, 512, 100, 256, 1), skip_layer=2)
SPECS = {"c1": di.C1_SPEC, "deepsdf": di.DEEPSDF_SPEC, "mixed": MIXED_SPEC}
_CTX = {}


def ctx_for(name):
    """The seeded decoder with nonzero biases, and its oracle."""
    if name not in _CTX:
        spec = SPECS[name]
        Ws, bs = di.make_decoder(spec, seed=5)
        rng = np.random.Generator(np.random.PCG64(6))
        bs = [(0.02 * rng.standard_normal(b.shape)).astype(np.float32) for b in bs]
        from oracle import dist_oracle as O
        _CTX[name] = (gpu_ctx(spec, Ws=Ws, bs=bs), O.Decoder(spec, Ws, bs))
    return _CTX[name]


# bounds of test_sdf_eval_*: FP32 2e-6, bf16 1e-3, split 1e-6 (x2 for the random biases' larger activations)
@pytest.mark.parametrize("prec,tol", [(0, 4e-6), (1, 2e-3), (2, 2e-6)], ids=["fp32", "bf16", "split"])
@pytest.mark.parametrize("name", list(SPECS))
def test_query_rows_do_not_depend_on_the_tile(name, prec, tol):
    from paper_1911_13225_amd import api
    ctx, dec = ctx_for(name)
    spec = SPECS[name]
    n = 256 * 128 + 1                        # full tiles and a rest on every CU
    rng = np.random.Generator(np.random.PCG64(7))
    P = rng.uniform(-0.7, 0.7, (n, 3)).astype(np.float32)
    Z = di.make_latents(3, spec.latent_dim, sigma=0.1)
    lat = (np.arange(n) % 3).astype(np.int32)
    Pt, lt, Zt = (torch.tensor(x, device="cuda") for x in (P, lat, Z))
    full = api.dist_sdf_eval(ctx, Pt, lt, Zt, prec)
    fo = dec.sdf(Z[lat[:300]].astype(np.float64), P[:300].astype(np.float64))
    assert np.abs(full[:300].cpu().numpy() - fo).max() <= tol
    for k in (1, 15, 16, 17, 31, 32, 33, 48, 49, 64, 65, 255 * 16 + 1, 256 * 16 + 1, 256 * 32 + 1, 256 * 48 + 1,
              256 * 64 + 1, 256 * 79):
        part = api.dist_sdf_eval(ctx, Pt[:k].contiguous(), lt[:k].contiguous(), Zt, prec)
        assert torch.equal(part, full[:k]), k


@pytest.mark.parametrize("n_lat", [1, 7, 8, 9, 33])
@pytest.mark.parametrize("name", list(SPECS))
def test_codes_fold_one_by_one(name, n_lat):
    """A code's folded biases do not depend on the codes beside it."""
    from paper_1911_13225_amd import api
    ctx, dec = ctx_for(name)
    Z = di.make_latents(n_lat, SPECS[name].latent_dim, sigma=0.1)
    P = np.random.Generator(np.random.PCG64(8)).uniform(-0.7, 0.7, (n_lat, 3)).astype(np.float32)
    Pt, Zt = torch.tensor(P, device="cuda"), torch.tensor(Z, device="cuda")
    f = api.dist_sdf_eval(ctx, Pt, torch.arange(n_lat, device="cuda", dtype=torch.int32), Zt, 0)
    assert np.abs(f.cpu().numpy() - dec.sdf(Z.astype(np.float64), P.astype(np.float64))).max() <= 4e-6
    for i in range(n_lat):
        one = api.dist_sdf_eval(ctx, Pt[i:i + 1].contiguous(), torch.zeros(1, device="cuda", dtype=torch.int32),
                                Zt[i:i + 1].contiguous(), 0)
        assert torch.equal(one, f[i:i + 1]), i


# Rays per CU from under one to over the tallest tile, so that the march fills
# its tiles to every height; K records, and a step limit that ends rays.
@pytest.mark.parametrize("prec", [0, 1, 2], ids=["fp32", "bf16", "split"])
@pytest.mark.parametrize("levels,k,steps", [(0, 1, 9), (1, 4, 50), (2, 3, 50)])
def test_march_does_not_depend_on_the_tile(prec, levels, k, steps):
    """An image's rays march the same alone, with few, and with many others."""
    from paper_1911_13225_amd import api
    spec = MIXED_SPEC
    ctx, _ = ctx_for("mixed")
    prm = di.TraceParams(max_steps=steps, c2f_levels=levels, k_samples=k, precision=prec, want_normals=0,
                         keep_history=1)
    z = torch.tensor(di.make_latents(1, spec.latent_dim, sigma=0.05), device="cuda")
    cams = di.random_sphere_cameras(48, 28, 36)
    g = torch.Generator(device="cuda").manual_seed(9)
    gd, gs = (torch.randn(1, 28, 36, generator=g, device="cuda") for _ in range(2))
    ref = None
    for n in (1, 9, 48):
        out = api.dist_render_fwd(ctx, cams[:n], z, prm, save=True)
        one = {key: out[key][:1].clone() for key in ("depth", "dist", "sil", "status", "nsteps", "queries")}
        gd_n, gs_n = torch.zeros_like(out["depth"]), torch.zeros_like(out["sil"])
        gd_n[:1], gs_n[:1] = gd * torch.isfinite(one["depth"]), gs        # seeds on the first image alone
        one["g_z"] = api.dist_render_bwd(ctx, out["saved"], gd_n, None, gs_n, n_latents=1)
        one["g_unrolled"] = api.dist_render_bwd_unrolled(ctx, out["saved"], gd_n, gs_n, n_latents=1)
        out["saved"].free()
        assert int(out["queries"].sum()) > 0
        if ref is None:
            ref = one
        for key in ref:
            # (48 images take the unrolled steps in smaller groups, and so add them in another order)
            assert (key == "g_unrolled" and n == 48) or torch.equal(ref[key], one[key]), (n, key)


# The weight gradient's rows run in chunks of 65,536 and each chunk's 64-row
# blocks in up to 8 (bf16) or 32 (float32) slices: fewer blocks than slices, in
# the only chunk and in the last one.
@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "bf16"])
@pytest.mark.parametrize("before,n", [(0, 1), (0, 64 * 3), (0, 64 * 41 + 5), (65536, 1), (65536, 64 * 5 + 3)])
def test_weight_gradient_slices(prec, before, n):
    """n samples behind `before` samples with zero seeds have the gradient of
    the n samples alone (in small groups, where every sum is short)."""
    from paper_1911_13225_amd import api
    ctx, _ = ctx_for("c1")
    rng = np.random.Generator(np.random.PCG64(11))
    P = torch.tensor(rng.uniform(-0.6, 0.6, (before + n, 3)).astype(np.float32), device="cuda")
    sd = torch.tensor(rng.standard_normal(before + n).astype(np.float32), device="cuda")
    sd[:before] = 0.0
    Z = torch.tensor(di.make_latents(1, 64, sigma=0.1), device="cuda")
    ids = torch.zeros(before + n, dtype=torch.int32, device="cuda")
    _, gW, gb = api.dist_sdf_vjp(ctx, P, ids, sd, Z, prec, want_theta=True)
    ref = None
    for i in range(before, before + n, 64):
        k = slice(i, min(i + 64, before + n))
        _, w, b = api.dist_sdf_vjp(ctx, P[k].contiguous(), ids[k].contiguous(), sd[k].contiguous(), Z, prec,
                                   want_theta=True)
        part = [x.double() for x in w + b]
        ref = part if ref is None else [x + y for x, y in zip(ref, part)]
    # both add the same float32 products, the one in sums of up to 256 rows and
    # their sums, the other in sums of 64: |difference| <= 256 ulp of the largest
    # sum of magnitudes, itself at most sqrt(n) times the (random-sign) sum's size
    for x, y in zip(gW + gb, ref):
        assert (x.double() - y).norm() <= 256 * 2.0 ** -24 * max(1.0, n ** 0.5) * y.norm()


@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "bf16"])
def test_unrolled_gradient_step_by_step_and_in_groups(prec):
    """Without the memory for a group of steps the gradient runs step by step.

    Both add the same float32 terms in different orders; a ray's adjoint passes
    through up to 50 roundings more in one than in the other, so 64 ulp of the
    gradient's norm bound the difference.
    """
    from paper_1911_13225_amd import api
    spec = di.C1_SPEC
    Ws, bs = di.make_decoder(spec, seed=5)
    prm = di.TraceParams(precision=prec, want_normals=0, keep_history=1)
    z = torch.tensor(di.make_latents(2, spec.latent_dim, sigma=0.05), device="cuda")
    cams = di.random_sphere_cameras(3, 44, 36)
    g = torch.Generator(device="cuda").manual_seed(10)
    gd, gs = (torch.randn(6, 44, 36, generator=g, device="cuda") for _ in range(2))
    grads, used = [], []
    for budget in (0, 24 << 20):
        ctx = api.Context.from_spec(spec, Ws, bs, hbm_budget=budget)
        free0 = torch.cuda.mem_get_info()[0]
        out = api.dist_render_fwd(ctx, cams, z, prm, save=True)
        seeds = gd * torch.isfinite(out["depth"])
        grads.append(api.dist_render_bwd_unrolled(ctx, out["saved"], seeds, gs, n_latents=2))
        again = api.dist_render_bwd_unrolled(ctx, out["saved"], seeds, gs, n_latents=2)
        torch.cuda.synchronize()
        used.append(free0 - torch.cuda.mem_get_info()[0])
        assert torch.equal(grads[-1], again)
        out["saved"].free()
        ctx.close()
    assert used[1] <= 24 << 20 < used[0]        # the second did run without the group's rows
    assert (grads[0] - grads[1]).norm() <= 64 * 2.0 ** -23 * grads[0].norm()


@pytest.mark.parametrize("prec", [0, 1, 2], ids=["fp32", "bf16", "split"])
@pytest.mark.parametrize("name", list(SPECS))
def test_tiles_of_one_latent_and_of_several(name, prec):
    """Layer 0 and the skip layer start on the matrix cores in a tile of one
    latent and on the vector units in a mixed one: the same bits either way, a
    latent that is not a number included (the ReLU of layer 0 makes it 0)."""
    from paper_1911_13225_amd import api
    ctx, _ = ctx_for(name)
    n = 256 * 128 + 70
    P = torch.tensor(np.random.Generator(np.random.PCG64(12)).uniform(-0.7, 0.7, (n, 3)).astype(np.float32),
                     device="cuda")
    Z = torch.tensor(di.make_latents(2, SPECS[name].latent_dim, sigma=0.1), device="cuda")
    Z[1] = Z[0]
    one = torch.zeros(n, device="cuda", dtype=torch.int32)
    two = (torch.arange(n, device="cuda") % 2).to(torch.int32)
    for k in (n, 33, 5):
        a = api.dist_sdf_eval(ctx, P[:k].contiguous(), one[:k].contiguous(), Z[:1].contiguous(), prec)
        b = api.dist_sdf_eval(ctx, P[:k].contiguous(), two[:k].contiguous(), Z, prec)
        assert torch.equal(a, b), k
    Z[:, 0] = float("nan")
    a = api.dist_sdf_eval(ctx, P, one, Z[:1].contiguous(), prec)
    b = api.dist_sdf_eval(ctx, P, two, Z, prec)
    assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(a.nan_to_num(), b.nan_to_num())


@pytest.mark.parametrize("shift", [0, 1], ids=["aligned", "shifted"])
@pytest.mark.parametrize("H,W", [(1, 3), (64, 64), (63, 65), (64, 65), (67, 71)])
def test_loss_of_odd_sizes_and_unaligned_maps(H, W, shift):
    """Maps whose sizes and addresses call for one or four pixels per access, of up to and over one
    4096-pixel run, and gradients written over the maps they come from.  A loss adds at most
    ceil(4757 / 1024) + 10 terms in a chain after about 8 roundings of each: 23 x 2^-24 < 2e-6 of the
    sum of absolute terms (the normals' at most w_n)."""
    from types import SimpleNamespace
    from oracle import dist_oracle as O
    from paper_1911_13225_amd import api, _native as N
    n, w = 2, (10.0, 1.0, 0.5)
    rng = np.random.default_rng(100 * H + W)
    maps = [rng.uniform(0.5, 2, (n, H, W)), rng.normal(size=(n, H, W, 3)), rng.normal(size=(n, H, W)),
            rng.uniform(0.5, 2, (n, H, W)), rng.normal(size=(n, H, W, 3)), rng.choice([0.0, 0.3, 1.0], (n, H, W))]
    for k in (1, 4):
        maps[k] /= np.linalg.norm(maps[k], axis=-1, keepdims=True)
    maps = [m.astype(np.float32) for m in maps]

    def dev(a):
        t = torch.empty(a.size + shift, device="cuda")[shift:].view(a.shape)
        t.copy_(torch.tensor(a))
        return t

    d, nr, s, dt, nt, st = [dev(a) for a in maps]
    loss, gd, gn, gs = api.dist_render_loss(d, nr, s, dt, nt, st, *w)
    for i in range(n):
        m = [a[i].astype(np.float64) for a in maps]
        r = SimpleNamespace(H=H, W=W, depth=m[0], normal=m[1], sil=m[2])
        L, g_d, g_n, g_s = O.loss_and_grads(r, *m[3:], w_d=w[0], w_s=w[1], w_n=w[2])
        L0 = O.loss_and_grads(r, *m[3:], w_d=w[0], w_s=w[1], w_n=0.0)[0]
        print(H, W, shift, i, float(loss[i]), L, flush=True)
        assert abs(float(loss[i]) - L) <= 2e-6 * (L0 + w[2])
        for got, want in ((gd, g_d), (gn, g_n), (gs, g_s)):
            np.testing.assert_allclose(got[i].cpu().numpy(), want, rtol=1e-6, atol=0)
    # the loss alone, and the gradients in the place of their maps
    assert torch.equal(loss, api.dist_render_loss(d, nr, s, dt, nt, st, *w, want_grad=False)[0])
    loss2 = torch.empty_like(loss)
    p = api._ptr
    api.check(N.load().dist_render_loss(n, H, W, p(d), p(nr), p(s), p(dt), p(nt), p(st), *w, p(loss2), p(d), p(nr),
                                        p(s), api._stream()))
    torch.cuda.synchronize()
    assert torch.equal(loss, loss2) and torch.equal(d, gd) and torch.equal(nr, gn) and torch.equal(s, gs)
