"""A hologram gives the same bits alone and in a batch, also where a rule that looks at
the size of the work lies between the two: the waves per tile of the rasterizer adjoint
(tiles per compute unit of one hologram against those of the batch) and the groups in
which focal planes are propagated (the memory of one hologram against the batch's)."""
import sys

import pytest
import torch

from paper_2511_15022_amd import binding, synth

pytestmark = pytest.mark.gpu

LAM = [639e-9, 515e-9, 473e-9]


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


def contexts(B, H, W, C, zs, n, **kw):
    """a batch and its holograms' own contexts, with optics that differ"""
    optics = [([LAM[(b + c) % 3] for c in range(C)], [z * (1 + 0.1 * b) for z in zs])
              for b in range(B)]
    pairs = kw.pop("max_pairs", 0)
    batch = binding.Context(H, W, C, 8e-6, *optics[0], max_gaussians=n, batch=B,
                            max_pairs=B * pairs, **kw)
    for b in range(B):
        batch.set_hologram_optics(b, *optics[b])
    return batch, [binding.Context(H, W, C, 8e-6, *o, max_gaussians=n, max_pairs=pairs, **kw)
                   for o in optics]


# up to 256 tiles alone (one per compute unit of 256) and 1024 together, 576 and 1152, and
# tiles of 8 x 8; the exponent's clamp needs a support beyond ten sigma
@pytest.mark.parametrize("B,H,W,C,n,kw", [
    (4, 256, 256, 1, 13107, {}),
    (4, 256, 256, 3, 6000, {}),
    (2, 384, 384, 1, 20000, {}),
    (4, 128, 128, 1, 3000, dict(tile=(8, 8))),
    (4, 256, 256, 1, 6000, dict(paper_alpha=True)),
    (4, 256, 256, 1, 500, dict(support_sigma=12.0, max_pairs=60000)),
])
def test_batch_equals_single_across_tile_counts(B, H, W, C, n, kw):
    say("batch bits", B, H, W, C, n, kw)
    batch, single = contexts(B, H, W, C, [2e-3], n, **kw)
    Ps = [binding.pack(synth.params(50 + b, n, H, W, C), device="cuda") for b in range(B)]
    Ts = [torch.from_numpy(synth.target(60 + b, C, H, W, L=1)).cuda() for b in range(B)]
    P, T = torch.cat(Ps), torch.stack(Ts, 1).contiguous()
    field = batch.rasterize(P, n)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    gf = torch.randn(field.shape, generator=gen, device="cuda", dtype=torch.complex64)
    adj = batch.rasterize_adjoint(P, n, gf)
    grads = batch.backward(P, n, field, T)
    m, v = torch.zeros_like(P), torch.zeros_like(P)
    batch.backward_step(P, n, field, T, m, v, 1, 1e-3)
    _, ok = batch.read_status()
    assert ok
    per = binding.param_count(n, C)
    for b, ctx in enumerate(single):
        mine = slice(b * per, (b + 1) * per)
        f1 = ctx.rasterize(Ps[b], n)
        assert torch.equal(field[b], f1)
        assert torch.equal(adj[mine], ctx.rasterize_adjoint(Ps[b], n, gf[b].contiguous())), b
        assert torch.equal(grads[mine], ctx.backward(Ps[b], n, f1, Ts[b])), b
        m1, v1 = torch.zeros_like(Ps[b]), torch.zeros_like(Ps[b])
        ctx.backward_step(Ps[b], n, f1, Ts[b], m1, v1, 1, 1e-3)
        assert torch.equal(P[mine], Ps[b]) and torch.equal(m[mine], m1) and torch.equal(v[mine], v1)


# three planes and more; pads whose columns split into four chains and into two, and one
# with no split.  Few Gaussians: the constant part of the default pair capacity holds the
# planes of one hologram and not those of eight; many: each hologram's own part holds them;
# in between: groups of two planes; and a pair capacity of the caller's
@pytest.mark.parametrize("H,W,pad,C,L,n,pairs", [
    (128, 128, (256, 256), 3, 3, 400, 0),
    (128, 128, (256, 256), 3, 3, 3276, 0),
    (64, 60, (128, 120), 1, 7, 800, 0),
    (45, 80, (90, 160), 2, 3, 60, 0),
    (45, 80, (90, 160), 2, 3, 60, 6000),
    (333, 40, (900, 90), 2, 4, 1300, 0),
    (50, 40, (75, 90), 1, 3, 30, 0),
])
def test_batch_equals_single_with_planes_in_groups(H, W, pad, C, L, n, pairs):
    B = 8
    say("batch bits, planes", H, W, pad, C, L, n, pairs)
    zs = [2e-3 + 5e-4 * l for l in range(L)]
    batch, single = contexts(B, H, W, C, zs, n, pad=pad, max_pairs=pairs)
    Ps = [binding.pack(synth.params(80 + b, n, H, W, C), device="cuda") for b in range(B)]
    P = torch.cat(Ps)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)
    T = torch.rand(L, B, C, H, W, generator=gen, device="cuda")
    gI = torch.randn(L, B, C, H, W, generator=gen, device="cuda")
    gu = torch.randn(L, B, C, H, W, generator=gen, device="cuda", dtype=torch.complex64)
    field = batch.rasterize(P, n)
    I, u = batch.propagate(field, intensity=True, field_out=True)
    adj, fadj = batch.propagate_adjoint(field, gI), batch.propagate_field_adjoint(gu)
    loss = torch.zeros(2 * B, dtype=torch.float64, device="cuda")
    gfield = torch.empty_like(field)
    grads = batch.backward(P, n, field, T, loss=loss, grad_field=gfield)
    per = binding.param_count(n, C)
    for b, ctx in enumerate(single):
        f1 = ctx.rasterize(Ps[b], n)
        assert torch.equal(field[b], f1)
        I1, u1 = ctx.propagate(f1, intensity=True, field_out=True)
        assert torch.equal(I[:, b], I1) and torch.equal(u[:, b], u1), b
        assert torch.equal(adj[b], ctx.propagate_adjoint(f1, gI[:, b].contiguous())), b
        assert torch.equal(fadj[b], ctx.propagate_field_adjoint(gu[:, b].contiguous())), b
        l1, g1 = torch.zeros_like(loss[:2]), torch.empty_like(f1)
        grads1 = ctx.backward(Ps[b], n, f1, T[:, b].contiguous(), loss=l1, grad_field=g1)
        assert torch.equal(gfield[b], g1) and torch.equal(grads[b * per:(b + 1) * per], grads1), b
        assert torch.equal(loss[2 * b:2 * b + 2], l1), b
