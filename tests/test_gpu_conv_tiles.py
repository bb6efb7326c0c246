"""The convolution's tile variants (rows per wave, channel blocks, weights in
registers or in LDS, one or two inputs, channel counts that are no multiple of
16) at the edges of their tiles, against nine shifted products in float64 of
the same BF16 inputs.

Tolerance.  A sum has at most 9 * 400 FP32 additions of rounded products that are
exact in FP32; its error grows as the square root of their number:
sqrt(3600) * 0.3 * 2^-24 = 1.1e-6 of the sum's scale for the longest, and the
relative L2 over an image is below that.  Bar: 2e-6.  BF16 outputs are the FP32 sum
rounded once: 2^-9 at most each."""
import ctypes
import sys

import pytest
import torch

from paper_2511_15022_amd import binding

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


def ptr(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def inputs(H, W, c1, up, c2, cout, seed=3):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    x1 = r(H >> up, W >> up, c1).bfloat16()
    x2 = r(H, W, c2).bfloat16() if c2 else None
    return x1, x2, r(cout, 9, c1 + c2).bfloat16(), r(cout)


def reference(x1, x2, w, b, up, H, W):
    x = x1.double()
    if up:
        x = x.repeat_interleave(2, 0).repeat_interleave(2, 1)
    if x2 is not None:
        x = torch.cat([x, x2.double()], -1)
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    y = b.double().expand(H, W, -1).clone()
    for t in range(9):
        ky, kx = divmod(t, 3)
        y += (xp[ky:ky + H, kx:kx + W].reshape(H * W, -1) @ w[:, t].double().T).reshape(H, W, -1)
    return y


CASES = [
    # (H, W, c1, up, c2, cout): at most 32 channels in, few tiles; partial tiles each way
    (9, 37, 24, 0, 0, 32), (5, 33, 8, 0, 0, 8), (1, 1, 32, 0, 0, 40),
    # the same with many tiles (four rows per wave)
    (251, 1003, 32, 0, 0, 24),
    # one input, few and many tiles, one and two channel blocks per wave
    (17, 31, 48, 0, 0, 32), (250, 1001, 48, 0, 0, 32), (250, 1001, 48, 0, 0, 64),
    # two inputs, the first upsampled
    (18, 70, 64, 1, 32, 32), (252, 1000, 32, 1, 32, 32), (258, 1006, 64, 1, 16, 128),
    # an upsampled input alone; channels that are no multiple of 16, also across the inputs
    (16, 34, 32, 1, 0, 32), (13, 65, 40, 0, 0, 24), (14, 40, 24, 1, 24, 16), (7, 33, 16, 0, 8, 48),
    (250, 1000, 40, 0, 24, 32), (30, 30, 56, 0, 0, 64),
    # the deepest sum
    (12, 40, 256, 1, 144, 64),
]


@pytest.mark.parametrize("H,W,c1,up,c2,cout", CASES)
def test_conv_tiles_match_float64(H, W, c1, up, c2, cout):
    say("conv", H, W, c1, up, c2, cout)
    x1, x2, w, b = inputs(H, W, c1, up, c2, cout)
    L = binding.lib()
    o32 = torch.full((H, W, cout), float("nan"), device="cuda")
    o16 = torch.zeros(H, W, cout, dtype=torch.bfloat16, device="cuda")
    binding._check(L.cgh_net_conv3x3(ptr(x1), c1, up, ptr(x2), c2, H, W, ptr(w), ptr(b), cout, 1,
                                     ptr(o32), ptr(o16), stream()))
    ref = reference(x1, x2, w, b, up, H, W)
    assert float((o32.double() - ref).norm() / ref.norm()) <= 2e-6
    assert torch.equal(o16, o32.clamp(min=0).bfloat16())


WGRAD = [
    # one tile and parts of one; shares of one and of several tiles; an upsampled first
    # input; blocks of 32 channels that straddle the two inputs or end early
    (5, 7, 8, 0, 0, 8), (16, 32, 32, 0, 0, 32), (33, 65, 24, 0, 0, 40), (18, 34, 40, 1, 24, 16),
    (70, 130, 64, 1, 32, 64), (250, 500, 32, 0, 0, 24), (40, 40, 256, 0, 0, 256),
]


@pytest.mark.parametrize("H,W,c1,up,c2,cout", WGRAD)
def test_weight_gradients_match_float64(H, W, c1, up, c2, cout):
    """Bar: sums of at most 125,000 exact products: sqrt(125000) * 0.3 * 2^-24 = 6e-6
    relative to the sum's scale if added one by one; the partial sums are shorter."""
    say("wgrad", H, W, c1, up, c2, cout)
    x1, x2, _, _ = inputs(H, W, c1, up, c2, cout)
    cin = c1 + c2
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    gy = torch.randn(H, W, cout, generator=g, device="cuda").bfloat16()
    L = binding.lib()
    nb = L.cgh_net_wgrad_workspace(H, W, cin, cout)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    gw = torch.empty(cout, 9, cin, device="cuda")
    gb = torch.empty(cout, device="cuda")
    for k in range(2):
        binding._check(L.cgh_net_conv3x3_wgrad(ptr(x1), c1, up, ptr(x2), c2, H, W, ptr(gy), cout,
                                               ptr(gw), ptr(gb), ptr(ws), nb, stream()))
        if k == 0:
            first = gw.clone()
    assert torch.equal(first, gw)
    x = x1.double()
    if up:
        x = x.repeat_interleave(2, 0).repeat_interleave(2, 1)
    if x2 is not None:
        x = torch.cat([x, x2.double()], -1)
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    g64 = gy.double().reshape(H * W, cout)
    ref = torch.stack([g64.T @ xp[t // 3:t // 3 + H, t % 3:t % 3 + W].reshape(H * W, cin)
                       for t in range(9)], 1)
    assert float((gw.double() - ref).norm() / ref.norm()) <= 6e-6
    assert float((gb.double() - g64.sum(0)).norm() / g64.sum(0).norm()) <= 6e-6


def test_wgrad_sums_of_many_layers():
    """The shares of several layers, summed in one call, give the values of the calls one
    by one: few and many shares, channels that are no multiple of 32, a missing bias,
    and more layers than one launch takes."""
    L = binding.lib()
    shapes = [(38, 70, 24, 40), (16, 32, 32, 32), (200, 264, 8, 8), (64, 64, 96, 32), (8, 8, 64, 128),
              (130, 100, 32, 64)]
    jobs, keep, want = [], [], []
    for k in range(19):
        H, W, cin, cout = shapes[k % len(shapes)]
        x, _, _, _ = inputs(H, W, cin, 0, 0, cout)
        gy = torch.randn(H, W, cout, device="cuda").bfloat16()
        out = lambda: (torch.full((cout, 9, cin), 7.0, device="cuda"),
                       torch.full((cout,), 7.0, device="cuda"))
        (gw, gb), (rw, rb) = out(), out()
        nb = L.cgh_net_wgrad_workspace(H, W, cin, cout)
        ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
        binding._check(L.cgh_net_conv3x3_wgrad(ptr(x), cin, 0, None, 0, H, W, ptr(gy), cout, ptr(rw),
                                               None if k == 3 else ptr(rb), ptr(ws), nb, stream()))
        ns = L.cgh_net_wgrad_shares_bytes(H, W, cin, cout)
        sh = torch.empty(ns, dtype=torch.uint8, device="cuda")
        assert L.cgh_net_wgrad_shares(ptr(x), cin, 0, None, 0, H, W, ptr(gy), cout, ptr(sh), ns - 1,
                                      stream()) != 0
        binding._check(L.cgh_net_wgrad_shares(ptr(x), cin, 0, None, 0, H, W, ptr(gy), cout, ptr(sh),
                                              ns, stream()))
        jobs.append(binding.cgh_net_wgrad_job(H, W, cin, cout, ptr(sh), ptr(gw),
                                              None if k == 3 else ptr(gb)))
        keep += [x, gy, ws, sh]
        want.append((gw, rw, gb, rb))
    say("wgrad sums", len(jobs))
    binding._check(L.cgh_net_wgrad_sums((binding.cgh_net_wgrad_job * len(jobs))(*jobs), len(jobs),
                                        stream()))
    for gw, rw, gb, rb in want:
        assert torch.equal(gw, rw) and torch.equal(gb, rb)


def test_fused_passes_equal_their_parts():
    """The pooled convolution, the gated input adjoint, the gated upsampling adjoint
    and the gated combination give the values of the separate calls."""
    say("fused passes")
    L = binding.lib()
    H, W, c, co = 38, 70, 48, 64
    x1, _, w, b = inputs(H, W, c, 0, 0, co)
    bf = lambda *s: torch.zeros(*s, dtype=torch.bfloat16, device="cuda")
    o, o2, p, p2 = bf(H, W, co), bf(H, W, co), bf(H // 2, W // 2, co), bf(H // 2, W // 2, co)
    chk = binding._check
    chk(L.cgh_net_conv3x3(ptr(x1), c, 0, None, 0, H, W, ptr(w), ptr(b), co, 1, None, ptr(o), stream()))
    chk(L.cgh_net_pool2(ptr(o), H, W, co, ptr(p), stream()))
    chk(L.cgh_net_conv3x3_pool2(ptr(x1), c, 0, None, 0, H, W, ptr(w), ptr(b), co, 1, ptr(o2), ptr(p2),
                                stream()))
    assert torch.equal(o, o2) and torch.equal(p, p2)
    gate = torch.randn(H, W, co, device="cuda").clamp(min=0).bfloat16()
    gate[0, 0, :3] = torch.tensor([float("inf"), float("nan"), -0.0])
    g32, z, z2 = torch.empty(H, W, co, device="cuda"), bf(H, W, co), bf(H, W, co)
    chk(L.cgh_net_conv3x3(ptr(x1), c, 0, None, 0, H, W, ptr(w), None, co, 0, ptr(g32), None, stream()))
    chk(L.cgh_net_relu_grad(ptr(g32), ptr(gate), g32.numel(), ptr(z), stream()))
    chk(L.cgh_net_conv3x3_gated(ptr(x1), c, H, W, ptr(w), co, ptr(gate), ptr(z2), stream()))
    assert torch.equal(z, z2)
    # the first 40 of 64 channels through the upsampling, the other 24 through the skip
    up, small = torch.empty(H // 2, W // 2, 40, device="cuda"), gate[:H // 2, :W // 2, :40].contiguous()
    y, y2 = bf(H // 2, W // 2, 40), bf(H // 2, W // 2, 40)
    chk(L.cgh_net_up_adjoint(ptr(g32), H, W, co, 40, ptr(up), stream()))
    chk(L.cgh_net_relu_grad(ptr(up), ptr(small), up.numel(), ptr(y), stream()))
    chk(L.cgh_net_up_adjoint_gated(ptr(g32), H, W, co, 40, ptr(small), ptr(y2), stream()))
    assert torch.equal(y, y2)
    gp = torch.randn(H // 2, W // 2, 24, device="cuda")
    act = gate[:, :, :24].contiguous()
    cmb, q, q2 = torch.empty(H, W, 24, device="cuda"), bf(H, W, 24), bf(H, W, 24)
    chk(L.cgh_net_grad_combine(ptr(gp), ptr(g32), co, 40, H, W, 24, ptr(cmb), stream()))
    chk(L.cgh_net_relu_grad(ptr(cmb), ptr(act), cmb.numel(), ptr(q), stream()))
    chk(L.cgh_net_grad_combine_gated(ptr(gp), ptr(g32), co, 40, H, W, 24, ptr(act), ptr(q2), stream()))
    assert torch.equal(q, q2)


# Images so wide that the rows of a tile lie further apart than 32-bit byte offsets reach
# (17 rows of 2^20 x 64 channels are 2.1 GB): one input, a skip of 136 channels beside an
# upsampled input, an upsampled input of 264 with a skip that shares its last block.
FAR_W = 1 << 20
FAR = [(18, 64, 0, 0, 8), (18, 8, 1, 136, 8), (18, 264, 1, 8, 16)]
WINDOWS = [(0, 70), (FAR_W // 2 - 36, FAR_W // 2 + 34), (FAR_W - 70, FAR_W)]


def far_inputs(H, c1, up, c2, cout):
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    bf = lambda *s: torch.empty(*s, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    return (bf(H >> up, FAR_W >> up, c1), bf(H, FAR_W, c2) if c2 else None, bf(cout, 9, c1 + c2),
            torch.randn(cout, generator=g, device="cuda"))


def window(x1, x2, up, a, b):
    """the inputs of columns a .. b - 1, two more on each side that has them"""
    lo, hi = max(0, a - 2), min(FAR_W, b + 2)
    return x1[:, lo >> up:hi >> up], None if x2 is None else x2[:, lo:hi], lo, hi


@pytest.mark.parametrize("H,c1,up,c2,cout", FAR)
def test_conv_of_far_rows_matches_float64(H, c1, up, c2, cout):
    """Bar: as above."""
    say("far conv", H, c1, up, c2, cout)
    x1, x2, w, bias = far_inputs(H, c1, up, c2, cout)
    o32 = torch.full((H, FAR_W, cout), float("nan"), device="cuda")
    o16 = torch.zeros(H, FAR_W, cout, dtype=torch.bfloat16, device="cuda")
    binding._check(binding.lib().cgh_net_conv3x3(
        ptr(x1), c1, up, ptr(x2), c2, H, FAR_W, ptr(w), ptr(bias), cout, 1, ptr(o32), ptr(o16),
        stream()))
    for a, b in WINDOWS:
        y1, y2, lo, hi = window(x1, x2, up, a, b)
        ref = reference(y1, y2, w, bias, up, H, hi - lo)[:, a - lo:b - lo]
        got = o32[:, a:b].double()
        # each row on its own: a wrong row cannot hide in the others' norm
        err = (got - ref).norm(dim=(1, 2)) / ref.norm(dim=(1, 2))
        assert float(err.max()) <= 2e-6, (a, err.tolist())
    assert torch.equal(o16, o32.clamp(min=0).bfloat16())


@pytest.mark.parametrize("H,c1,up,c2,cout", [(18, 8, 1, 72, 8), (18, 264, 1, 8, 8), (18, 8, 0, 0, 72)])
def test_weight_gradients_of_far_rows_match_float64(H, c1, up, c2, cout):
    """dL/dout is zero outside the windows, so that the sums run over them alone (3780
    products); bar as for the weight gradients above."""
    say("far wgrad", H, c1, up, c2, cout)
    x1, x2, _, _ = far_inputs(H, c1, up, c2, cout)
    L, cin = binding.lib(), c1 + c2
    gy = torch.zeros(H, FAR_W, cout, dtype=torch.bfloat16, device="cuda")
    gw, gb = torch.empty(cout, 9, cin, device="cuda"), torch.empty(cout, device="cuda")
    want, want_b = torch.zeros(cout, 9, cin, dtype=torch.double, device="cuda"), 0
    for a, b in WINDOWS:
        gy[:, a:b] = torch.randn(H, b - a, cout, device="cuda").bfloat16()
        y1, y2, lo, hi = window(x1, x2, up, a, b)
        x = y1.double()
        if up:
            x = x.repeat_interleave(2, 0).repeat_interleave(2, 1)
        if y2 is not None:
            x = torch.cat([x, y2.double()], -1)
        xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
        g64 = gy[:, a:b].double().reshape(-1, cout)
        want += torch.stack(
            [g64.T @ xp[t // 3:t // 3 + H, a - lo + t % 3:b - lo + t % 3].reshape(-1, cin)
             for t in range(9)], 1)
        want_b = want_b + g64.sum(0)
    nb = L.cgh_net_wgrad_shares_bytes(H, FAR_W, cin, cout)
    sh = torch.empty(nb, dtype=torch.uint8, device="cuda")
    binding._check(L.cgh_net_wgrad_shares(ptr(x1), c1, up, ptr(x2), c2, H, FAR_W, ptr(gy), cout,
                                          ptr(sh), nb, stream()))
    job = binding.cgh_net_wgrad_job(H, FAR_W, cin, cout, ptr(sh), ptr(gw), ptr(gb))
    binding._check(L.cgh_net_wgrad_sums((binding.cgh_net_wgrad_job * 1)(job), 1, stream()))
    assert float((gw.double() - want).norm() / want.norm()) <= 6e-6
    assert float((gb.double() - want_b).norm() / want_b.norm()) <= 6e-6
