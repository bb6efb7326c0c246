"""The rasterizer adjoint's walk over two pixels of a row at a time, for every tile
shape and channel count, where its boxes are odd: Gaussians one to three pixels wide,
some beside tile and canvas edges (the box grows by a column on the side that has
room), and some that fill whole tiles.

Tolerance: the pair sums are FP32 sums of at most 256 products per tile, 3e-7 of the
sum of the terms' sizes; more comes from the FP32 geometry, whose inverse covariance
of a Gaussian with axes 12 : 1 (condition 144) is off by about 3 * 144 * 2^-24 = 3e-5,
times the exponent, up to 6.5 at the rim of the support: 2e-4 there.  The bar for a
whole parameter group is 3e-4."""
import sys

import numpy as np
import pytest
import torch

from paper_2511_15022_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", binding.TILE_SHAPES)
@pytest.mark.parametrize("H,W,C", [(43, 71, 1), (43, 71, 2), (43, 71, 3), (43, 71, 4),
                                   (450, 460, 3)])  # few tiles (8 waves each), many (3)
def test_odd_boxes_match_oracle(O, tile, H, W, C):
    print("[gpu-case] adjoint boxes", tile, H, W, C, flush=True)
    sys.stdout.flush()
    n = 240
    lam = [639e-9, 515e-9, 473e-9, 450e-9][:C]
    p = synth.params(5, n, H, W, C)
    rng = np.random.default_rng(6)
    # means on a grid of tile corners, up to 1.5 pixels off; two scales in 0.15 .. 12
    x = np.clip(rng.integers(0, W // 8 + 1, n) * 8 + rng.uniform(-1.5, 1.5, n), 0.2, W - 0.2)
    y = np.clip(rng.integers(0, H // 8 + 1, n) * 8 + rng.uniform(-1.5, 1.5, n), 0.2, H - 0.2)
    dt = p["mean_pre"].dtype
    p["mean_pre"] = np.arctanh(np.stack([2 * x / W - 1, 2 * y / H - 1], -1)).astype(dt)
    p["log_scale"] = np.where(rng.random((n, 1)) < 0.7, rng.uniform(-3.0, -0.5, (n, 2)),
                              rng.uniform(0.0, 2.5, (n, 2))).astype(dt)
    pad = (90, 144) if H == 43 else (900, 960)
    opt = O.Optics(H, W, C, *pad, 8e-6, lam, [2e-3])
    ctx = binding.Context(H, W, C, 8e-6, lam, [2e-3], pad=pad,
                          max_gaussians=n, max_pairs=64 * n, tile=tile)
    ref = O.forward_backward(p, synth.target(7, C, H, W), opt)
    P = binding.pack(p, device="cuda")
    ctx.rasterize(P, n)
    gf = torch.from_numpy(ref["grad_field"].astype(np.complex64)).cuda()
    g = binding.unpack(ctx.rasterize_adjoint(P, n, gf).cpu(), n, C)
    for k in binding.PARAM_KEYS:
        a, b = g[k].numpy(), ref["grads"][k]
        err = np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel())
        print("[gpu-case]", k, err, flush=True)
        assert err <= 3e-4, (k, err)


@pytest.mark.parametrize("mode", ["paper_alpha", "clamp"])
@pytest.mark.parametrize("tile", binding.TILE_SHAPES)
@pytest.mark.parametrize("H,W,C", [(43, 71, 1), (43, 71, 3), (450, 460, 3)])  # few tiles, many
def test_odd_boxes_in_other_weights_match_oracle(O, mode, tile, H, W, C):
    """The same walk with the Alg. 2 weight (its own limits of the exponent and its clamp
    sum) and with a support so wide that the exponent's clamp is active inside it.

    Tolerance: 2e-4 from the geometry, as above (terms with a larger exponent than 6.5
    weigh e^-6.5 and less); with the Alg. 2 weight, a pair that rounding puts on the other
    side of the skip or of the clamp moves single terms by 1/255 of a pixel's, of some
    thousands.  Bar: 1e-3."""
    print("[gpu-case] adjoint boxes", mode, tile, H, W, C, flush=True)
    sys.stdout.flush()
    n = 240
    pa = mode == "paper_alpha"
    k = 3.0 if pa else 12.0
    lam = [639e-9, 515e-9, 473e-9][:C]
    p = synth.params(15, n, H, W, C)
    rng = np.random.default_rng(16)
    x = np.clip(rng.integers(0, W // 8 + 1, n) * 8 + rng.uniform(-1.5, 1.5, n), 0.2, W - 0.2)
    y = np.clip(rng.integers(0, H // 8 + 1, n) * 8 + rng.uniform(-1.5, 1.5, n), 0.2, H - 0.2)
    dt = p["mean_pre"].dtype
    p["mean_pre"] = np.arctanh(np.stack([2 * x / W - 1, 2 * y / H - 1], -1)).astype(dt)
    p["log_scale"] = np.where(rng.random((n, 1)) < 0.7, rng.uniform(-3.0, -0.5, (n, 2)),
                              rng.uniform(0.0, 2.0, (n, 2))).astype(dt)
    if pa:
        # some nearly opaque: alpha G > 0.99 at the pixels nearest to their means
        p["opacity_pre"] = rng.uniform(-4.0, 9.0, n).astype(np.float32)
    pad = (90, 144) if H == 43 else (900, 960)
    opt = O.Optics(H, W, C, *pad, 8e-6, lam, [2e-3], k=k, flags=O.FLAG_PAPER_ALPHA if pa else 0)
    ctx = binding.Context(H, W, C, 8e-6, lam, [2e-3], pad=pad, support_sigma=k, paper_alpha=pa,
                          max_gaussians=n, max_pairs=2000 * n, tile=tile)
    ref = O.forward_backward(p, synth.target(17, C, H, W), opt)
    P = binding.pack(p, device="cuda")
    ctx.rasterize(P, n)
    _, ok = ctx.read_status()
    assert ok
    gf = torch.from_numpy(ref["grad_field"].astype(np.complex64)).cuda()
    g = binding.unpack(ctx.rasterize_adjoint(P, n, gf).cpu(), n, C)
    for key in binding.PARAM_KEYS:
        a, b = g[key].numpy(), ref["grads"][key]
        err = np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel())
        print("[gpu-case]", key, err, flush=True)
        assert err <= 1e-3, (key, err)
