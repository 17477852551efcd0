"""The pack kernel's loads: rows that start at every byte alignment, sources that
do not start on a word, the tensor's last bytes, rows on both sides of what is
read by bytes and tensors on both sides of what takes 128-channel tiles, against
the oracle; and the largest grid of 64-channel tiles."""
import numpy as np
import pytest

import oracle
from _util import announce, assert_same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,c,h,w", [(1, 8, 1, 31), (2, 8, 1, 33), (1, 64, 5, 7), (3, 72, 7, 9), (1, 136, 1, 129),
                                     (2, 16, 13, 5), (1, 8, 1, 1), (5, 200, 3, 3), (5, 200, 2, 5), (5, 200, 1, 11),
                                     (60, 256, 29, 33), (72, 256, 29, 33), (140, 160, 23, 21)])
@pytest.mark.parametrize("bits,signed", [(4, False), (4, True), (8, True)])
def test_pack_unaligned_rows(n, c, h, w, bits, signed):
    import torch
    from paper_2202_06819_amd import qconv as q

    g = np.random.default_rng([91, n, c, h, w, bits, signed])
    x = g.integers(-128, 128, size=(n, c, h, w)).astype(np.int8)
    want = oracle.relayout_pack(x, bits, signed)
    for shift in (0, 1, 3, 6):
        announce(f"pack {n}x{c}x{h}x{w} {bits}-bit, source {shift} bytes past a word")
        buf = torch.zeros(x.size + shift, dtype=torch.int8, device="cuda:0")
        src = buf[shift:].view(n, c, h, w)
        src.copy_(torch.from_numpy(x))
        y = q.pack(src, bits, signed)
        torch.cuda.synchronize()
        assert_same(y.cpu().numpy(), want, f"pack {n}x{c}x{h}x{w} {bits} {shift}")


def test_pack_of_the_largest_grid():
    """A launch holds fewer than 2^32 threads: nine million one-pixel images of 132
    channels are 27 million workgroups of 128.  One pixel an image, the packed
    layout is the source's."""
    import torch
    from paper_2202_06819_amd import qconv as q

    x = torch.randint(-128, 128, (9_000_000, 132, 1, 1), dtype=torch.int8, device="cuda:0")
    announce("pack 9000000x132x1x1 8-bit")
    y = q.pack(x, 8, True)
    torch.cuda.synchronize()
    assert torch.equal(y.view(-1), x.view(-1))


def test_pack_beyond_the_largest_launch():
    """34 million one-pixel images are as many workgroups of 128 threads, more than
    the 2^32 threads a launch counts: the pack on its own, and the one that
    qconv2d_packing runs before a convolution of several stages.  One pixel an
    image, the packed layout is the source's and only the centre taps count."""
    import torch
    from paper_2202_06819_amd import qconv as q

    n, c, k, shift = 34_000_000, 16, 4, 22
    d = dict(n=n, h=1, w=1, c=c, k=k, r=3, s=3, stride_h=1, stride_w=1, pad_h=1, pad_w=1, bits=8, x_signed=1, w_signed=1)
    tile = next(t["id"] for t in q.tiles() if t["variant"] == 2 and q.tile_status(d, t["id"]) == 0)
    g = torch.Generator(device="cuda:0").manual_seed(93)
    x = torch.randint(-128, 128, (n, c, 1, 1), dtype=torch.int8, device="cuda:0", generator=g)
    w = torch.randint(-127, 128, (k, c, 3, 3), dtype=torch.int8, device="cuda:0", generator=g)
    mult = torch.randint(1 << 14, 1 << 15, (k,), dtype=torch.int32, device="cuda:0", generator=g)
    announce("pack 34000000x16x1x1 8-bit")
    y = q.pack(x, 8, True)
    torch.cuda.synchronize()
    assert torch.equal(y.view(-1), x.view(-1))
    del y
    announce("fused pack 34000000x16x1x1 8-bit")
    call = q.PackingConv2dCall(d, x, q.prepare_filters(d, q.pack(w, 8, True), tile), tile=tile, mult=mult, shift=shift,
                               relu=False, clamp=(-128, 127), x_packed=True)
    y = call().view(n, k)
    torch.cuda.synchronize()
    assert torch.equal(call.x_packed.view(-1), x.view(-1))
    centre = w[:, :, 1, 1].double().t().contiguous()
    for i in range(0, n, 4_000_000):
        acc = (x[i:i + 4_000_000].view(-1, c).double() @ centre).to(torch.int64)
        want = ((acc * mult.to(torch.int64) + (1 << (shift - 1))) >> shift).clamp(-128, 127).to(torch.int8)
        assert torch.equal(y[i:i + 4_000_000], want)
