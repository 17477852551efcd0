"""The pack kernel's loads: rows that start at every byte alignment, sources that
do not start on a word, and the tensor's last bytes, against the oracle."""
import numpy as np
import pytest

import oracle
from _util import announce, assert_same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,c,h,w", [(1, 8, 1, 31), (2, 8, 1, 33), (1, 64, 5, 7), (3, 72, 7, 9), (1, 136, 1, 129),
                                     (2, 16, 13, 5), (1, 8, 1, 1)])
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
