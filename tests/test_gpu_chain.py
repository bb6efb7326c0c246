"""The chain FFT passes at the lengths where they can go wrong, against the FP64
oracle: the smallest and longest chains of each split, chains that leave lanes
idle or need several butterflies per lane, canvases smaller than half the
padded grid, and grids whose last column tile is partly empty.

Tolerance.  A propagation is four transforms of at most 13 radix-2 levels; each
level rounds its values about three times to a relative 2^-24 (the rms of a
rounding is 0.3 of that), the errors are independent, and twiddles and transfer
values carry one rounding each: sqrt(4 (13 * 3 + 2)) * 0.3 * 2^-24 = 2.3e-7
relative L2.  The bar is four times that, 1e-6; for gradients, which add the
loss's own arithmetic on two propagations, 4e-6."""
import sys

import numpy as np
import pytest
import torch

from paper_2511_15022_amd import binding

pytestmark = pytest.mark.gpu

TOL = 1e-6
GRAD_TOL = 4e-6


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


def rel(a, b):
    return float(np.linalg.norm((np.asarray(a) - b).ravel()) / np.linalg.norm(np.asarray(b).ravel()))


CASES = [
    # (H, W, Hp, Wp, C): chains of four, 16 x 16 (the shortest) and with idle samples
    (32, 32, 64, 64, 1),
    (21, 19, 64, 72, 2),
    # chains of two (padded lengths 2 M, M odd), partly empty last tile
    (25, 27, 50, 54, 1),
    (220, 131, 450, 270, 1),
    # several butterflies per lane, odd canvases
    (333, 517, 720, 1080, 1),
    (128, 128, 256, 512, 1),
    # one stage of radix 25 or 27 in the fused butterfly; the longest columns
    (600, 9, 1250, 64, 2),
    (1215, 11, 2430, 64, 1),
    (2400, 8, 4800, 64, 1),
    # the longest rows of each split
    (7, 4096, 64, 8192, 1),
    (5, 3645, 64, 7290, 1),
    (6, 3000, 64, 6250, 1),
    # two and four column chains per wave, with and without idle lanes, padded layouts in
    # LDS; the last short chain and the first long one; the longest power of two
    (500, 33, 1000, 72, 1),
    (600, 12, 1200, 64, 1),
    (640, 20, 1280, 64, 1),
    (1280, 9, 2560, 64, 1),
    (449, 16, 900, 64, 1),
    (486, 16, 972, 64, 1),
    (2048, 8, 4096, 64, 1),
    # two planes: the adjoint column pass adds into its destination
    (45, 80, 90, 160, 3),
]


@pytest.mark.parametrize("H,W,Hp,Wp,C", CASES)
def test_chain_passes_match_oracle(O, H, W, Hp, Wp, C):
    zs = [2e-3, -1e-3] if C == 3 else [2e-3]
    L = len(zs)
    lambdas = [639e-9, 515e-9, 473e-9][:C]
    say("chain", H, W, Hp, Wp, C, L)
    opt = O.Optics(H, W, C, Hp, Wp, 8e-6, lambdas, zs)
    ctx = binding.Context(H, W, C, 8e-6, lambdas, zs, pad=(Hp, Wp), max_gaussians=1)
    rng = np.random.default_rng(5)
    f = (rng.standard_normal((C, H, W)) + 1j * rng.standard_normal((C, H, W))).astype(np.complex64)
    F = torch.from_numpy(f).cuda()
    I, u = ctx.propagate(F, intensity=True, field_out=True)
    ref = O.propagate(f.astype(np.complex128), opt)
    assert rel(u.cpu().numpy(), ref) <= TOL
    assert rel(I.cpu().numpy(), np.abs(ref) ** 2) <= TOL
    gu = (rng.standard_normal((L, C, H, W)) + 1j * rng.standard_normal((L, C, H, W))).astype(
        np.complex64)
    g = ctx.propagate_field_adjoint(torch.from_numpy(gu).cuda())
    assert rel(g.cpu().numpy(), O.propagate_adjoint(gu.astype(np.complex128), opt)) <= TOL
    # the middle pass with the loss weights and its partial sums
    T = rng.random((L, C, H, W)).astype(np.float32)
    mask = (rng.random((L, H, W)) < 0.5).astype(np.float32)
    P = torch.zeros(6 + 2 * C, device="cuda")
    ctx.rasterize(P, 1)
    loss = torch.zeros(2, dtype=torch.float64, device="cuda")
    gf = torch.empty_like(F)
    ctx.backward(P, 1, F, torch.from_numpy(T).cuda(), loss=loss, grad_field=gf,
                 mask=torch.from_numpy(mask).cuda())
    w = 1.0 + mask[:, None].astype(np.float64) ** 2 + T.astype(np.float64) ** 2
    d = np.abs(ref) ** 2 - T
    assert abs(loss[0].item() - np.mean(w * d * d)) <= GRAD_TOL * np.mean(w * d * d)
    seed = 4.0 * w * d * ref / d.size
    assert rel(gf.cpu().numpy(), O.propagate_adjoint(seed, opt)) <= GRAD_TOL


def test_transfer_table_follows_the_optics():
    """get_transfer of a chain context is the table of a context made with the
    same optics, after set_optics too (bitwise: the same kernel)."""
    a = binding.Context(45, 80, 2, 8e-6, [639e-9, 515e-9], [2e-3], max_gaussians=1)
    b = binding.Context(45, 80, 2, 8e-6, [473e-9, 639e-9], [-3e-3], max_gaussians=1)
    say("transfer table")
    assert not torch.equal(a.get_transfer(1, 0), b.get_transfer(1, 0))
    a.set_optics([473e-9, 639e-9], [-3e-3])
    for ch in range(2):
        assert torch.equal(a.get_transfer(ch, 0), b.get_transfer(ch, 0))


PIPED = [
    # (H, W, Hp, Wp, C): rows of two workgroups per CU and one, whose forward pass takes
    # several rows per workgroup; fewer rows than workgroups, and a remainder of rows
    (5, 2600, 64, 5400, 1),
    (257, 2700, 540, 5400, 2),
    (181, 4000, 384, 8000, 3),
    (523, 3645, 1080, 7290, 1),
]


@pytest.mark.parametrize("H,W,Hp,Wp,C", PIPED)
def test_long_rows_match_oracle(O, H, W, Hp, Wp, C):
    say("long rows", H, W, Hp, Wp, C)
    lam = [639e-9, 515e-9, 473e-9][:C]
    rng = np.random.default_rng(3)
    f = (rng.standard_normal((C, H, W)) + 1j * rng.standard_normal((C, H, W))).astype(np.complex64)
    opt = O.Optics(H, W, C, Hp, Wp, 8e-6, lam, [2e-3])
    ctx = binding.Context(H, W, C, 8e-6, lam, [2e-3], pad=(Hp, Wp), max_gaussians=16)
    _, u = ctx.propagate(torch.from_numpy(f).cuda(), intensity=True, field_out=True)
    assert rel(u.cpu().numpy(), O.propagate(f.astype(np.complex128), opt)) <= TOL


PLANES = [
    # (H, W, Hp, Wp, C, L, pairs): all planes in one pass, with the next plane's columns
    # loaded ahead (short last radices) and not; chains of two
    (45, 80, 90, 160, 3, 3, 0),
    (180, 96, 360, 192, 1, 2, 0),
    (333, 40, 900, 90, 2, 3, 0),
    (75, 75, 150, 150, 1, 8, 0),
    # little memory for the pairs: groups of 1, 1 and 1 planes, and of 2, 2, 2 and 1
    (90, 200, 180, 400, 2, 3, 64),
    (60, 64, 120, 128, 1, 7, 3000),
    # a last radix too long for the shared pass, and shapes with no chain split
    (600, 9, 1250, 64, 2, 3, 0),
    (50, 40, 75, 90, 1, 3, 0),
    (40, 60, 90, 90, 2, 2, 0),
]


@pytest.mark.parametrize("H,W,Hp,Wp,C,L,pairs", PLANES)
def test_planes_match_oracle(O, H, W, Hp, Wp, C, L, pairs):
    say("planes", H, W, Hp, Wp, C, L, pairs)
    zs = [2e-3 - 7e-4 * l for l in range(L)]
    lam = [639e-9, 515e-9, 473e-9][:C]
    opt = O.Optics(H, W, C, Hp, Wp, 8e-6, lam, zs)
    ctx = binding.Context(H, W, C, 8e-6, lam, zs, pad=(Hp, Wp), max_gaussians=1, max_pairs=pairs)
    rng = np.random.default_rng(11)
    cplx = lambda *s: (rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(np.complex64)
    f, gu = cplx(C, H, W), cplx(L, C, H, W)
    F = torch.from_numpy(f).cuda()
    I, u = ctx.propagate(F, intensity=True, field_out=True)
    ref = O.propagate(f.astype(np.complex128), opt)
    for l in range(L):
        assert rel(u[l].cpu().numpy(), ref[l]) <= TOL
    assert rel(I.cpu().numpy(), np.abs(ref) ** 2) <= TOL
    g = ctx.propagate_field_adjoint(torch.from_numpy(gu).cuda())
    assert rel(g.cpu().numpy(), O.propagate_adjoint(gu.astype(np.complex128), opt)) <= TOL
    gi = rng.random((L, C, H, W)).astype(np.float32)
    g = ctx.propagate_adjoint(F, torch.from_numpy(gi).cuda())
    assert rel(g.cpu().numpy(), O.propagate_adjoint(2.0 * gi * ref, opt)) <= GRAD_TOL
    T = rng.random((L, C, H, W)).astype(np.float32)
    mask = (rng.random((L, H, W)) < 0.5).astype(np.float32)
    P = torch.zeros(6 + 2 * C, device="cuda")
    ctx.rasterize(P, 1)
    loss = torch.zeros(2, dtype=torch.float64, device="cuda")
    gf = torch.empty_like(F)
    ctx.backward(P, 1, F, torch.from_numpy(T).cuda(), loss=loss, grad_field=gf,
                 mask=torch.from_numpy(mask).cuda())
    w = 1.0 + mask[:, None].astype(np.float64) ** 2 + T.astype(np.float64) ** 2
    d = np.abs(ref) ** 2 - T
    assert abs(loss[0].item() - np.mean(w * d * d)) <= GRAD_TOL * np.mean(w * d * d)
    assert rel(gf.cpu().numpy(), O.propagate_adjoint(4.0 * w * d * ref / d.size, opt)) <= GRAD_TOL


@pytest.mark.parametrize("H,W,Hp,Wp,C,L", [c[:6] for c in PLANES if c[6] == 0 and c[5] > 2])
def test_planes_together_match_oracle(O, H, W, Hp, Wp, C, L):
    """The same with room for all planes at once in the pairs' memory."""
    test_planes_match_oracle(O, H, W, Hp, Wp, C, L, 65536)


@pytest.mark.parametrize("H,W,Hp,Wp", [(45, 80, 90, 160), (64, 64, 128, 128), (50, 40, 75, 90)])
def test_get_transfer_reads_the_table_of_the_column_pass(H, W, Hp, Wp):
    """An entry changed in the workspace shows in get_transfer, and no other does: the
    column-major, scaled table of the chain passes and the row-major one of the others."""
    say("transfer table in the workspace", H, W, Hp, Wp)
    ctx = binding.Context(H, W, 1, 8e-6, [515e-9], [2e-3], pad=(Hp, Wp), max_gaussians=1)
    before = ctx.get_transfer()
    w = ctx.workspace[:ctx.workspace.numel() // 8 * 8].view(torch.complex64)
    chain = Hp % 2 == 0
    rows = before.T.contiguous() / (Hp * Wp) if chain else before
    first = rows.reshape(-1)[:8]
    hit = torch.ones(w.numel() - 8, dtype=torch.bool, device="cuda")
    for k in range(8):
        hit &= (w[k:w.numel() - 8 + k] - first[k]).abs() <= 1e-6 * first[k].abs()
    at = hit.nonzero().reshape(-1).tolist()
    assert len(at) == 1, at
    w[at[0] + 3] *= 2
    after = ctx.get_transfer()
    y, x = (3, 0) if chain else (0, 3)
    assert abs(after[y, x].item() - 2 * before[y, x].item()) <= 1e-6
    after[y, x] = before[y, x]
    assert torch.equal(after, before)


def test_get_transfer_is_unscaled_to_the_last_bit():
    """The scaled, column-major table gives the values of the row-major one: the same
    padded grid with a canvas that splits into chains and with one that does not."""
    say("transfer table, both layouts")
    a, b = (binding.Context(H, 80, 1, 8e-6, [515e-9], [2e-3], pad=(90, 160), max_gaussians=1,
                            aperture=70.0) for H in (45, 80))
    ta, tb = a.get_transfer(), b.get_transfer()
    assert torch.equal(ta, tb) and 0 < int((ta != 0).sum()) < ta.numel()
