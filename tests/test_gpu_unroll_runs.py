"""Patch unrolling on both sides of the rule that picks its kernel: runs (filter
columns x channels) of 15, 16 and 17 bytes, runs that end inside an output vector,
output vectors per pixel that do and do not divide a workgroup, rows wider than
one, and padding on every side, against the definition written out with numpy."""
import numpy as np
import pytest

from _util import announce, unroll_def

pytestmark = pytest.mark.gpu

# n, c, h, w, c_out, taps_h, stride_h, pad_h, taps_w, stride_w, pad_w
CASES = [
    (2, 3, 5, 9, 16, 1, 1, 0, 5, 1, 2),        # a run of 15
    (2, 4, 5, 9, 16, 1, 1, 0, 4, 1, 1),        # 16, all of the vector
    (1, 17, 3, 4, 32, 1, 1, 0, 1, 1, 0),       # 17, one column
    (2, 3, 11, 13, 64, 2, 2, 3, 7, 2, 3),      # two runs of 21 and zeros after them
    (1, 3, 11, 13, 48, 2, 1, 1, 7, 1, 3),      # three vectors a pixel: 256 % 3 != 0
    (1, 5, 6, 300, 256, 7, 1, 3, 7, 3, 2),     # rows wider than a workgroup, 16 vectors
    (3, 16, 2, 1, 4096, 2, 1, 1, 1, 1, 0),     # 256 vectors a pixel, one pixel a row
    (1, 1, 1, 16, 16, 1, 1, 0, 16, 1, 0),      # the smallest: one output vector
]


@pytest.mark.parametrize("n,c,h,w,c_out,th,sh,ph,tw,sw,pw", CASES)
def test_unroll_runs(n, c, h, w, c_out, th, sh, ph, tw, sw, pw):
    import torch
    from paper_2202_06819_amd import qconv as q

    announce(f"unroll {n}x{c}x{h}x{w} -> {c_out}, {th}x{tw}")
    x = np.random.default_rng([92, n, c, h, w, c_out]).integers(-128, 128, size=(n, c, h, w)).astype(np.int8)
    plan = dict(taps_h=th, stride_h=sh, pad_h=ph, out_h=(h + 2 * ph - th) // sh + 2, taps_w=tw, stride_w=sw, pad_w=pw)
    y = q.unroll(torch.from_numpy(x).to("cuda:0"), c_out, **plan)
    assert np.array_equal(y.cpu().numpy(), unroll_def(x, c_out, **plan))


@pytest.mark.parametrize("c,taps_w", [(1, 16), (16, 1), (1, 8)])
def test_unroll_beyond_the_largest_launch(c, taps_w):
    """17 million rows are as many workgroups of 256 threads, more than the 2^32
    threads a launch counts; both kernels.  A row of one pixel unrolls to its own
    bytes, channels after columns, and zeros."""
    import torch
    from paper_2202_06819_amd import qconv as q

    n = 17_000_000
    announce(f"unroll {n}x{c}x1x{taps_w}")
    x = torch.randint(-128, 128, (n, c, 1, taps_w), dtype=torch.int8, device="cuda:0")
    y = q.unroll(x, 16, taps_h=1, stride_h=1, pad_h=0, out_h=1, taps_w=taps_w, stride_w=1, pad_w=0).view(n, 16)
    torch.cuda.synchronize()
    real = c * taps_w
    assert torch.equal(y[:, :real].reshape(-1), x.view(-1)) and not y[:, real:].any()
