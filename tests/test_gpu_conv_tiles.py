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
