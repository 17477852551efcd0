"""Prepared layers that the library moves to the direct kernels by itself: small
layers at the edges of their tiles (pixel fragments, channel pairs and chunks,
padding wider than the filter, the end of the tensor) and every form of their
epilogue, from the filter image of every wide tile, against the oracle's sums.
Layers this small take the depth form with one round of steps in flight;
test_gpu_direct_forms.py names every form in turn."""
import numpy as np
import pytest

import oracle
import qconv_inputs as qi
from _util import announce, assert_same, epilogue_forms, oracle_threads, packed_values, requantised

pytestmark = pytest.mark.gpu

# (n, h, w, c, k, r, s, stride, pad, bits)
SHAPES = [
    (1, 1, 1, 32, 8, 1, 1, 1, 0, 4),        # one pixel, half a chunk
    (1, 3, 5, 64, 24, 1, 1, 1, 0, 4),       # 15 pixels
    (1, 4, 4, 96, 40, 1, 1, 1, 0, 4),       # 16 pixels, a chunk and a half: the last load ends at the tensor's end
    (1, 1, 17, 160, 72, 1, 1, 1, 0, 4),     # 17 pixels
    (3, 9, 7, 256, 64, 1, 1, 1, 0, 4),
    (2, 11, 5, 512, 136, 1, 1, 1, 0, 4),    # eight steps, all in flight
    (2, 9, 9, 128, 32, 1, 1, 2, 0, 4),      # strided 1x1
    (1, 7, 7, 32, 64, 3, 3, 1, 1, 4),       # half a chunk under a 3x3
    (2, 7, 18, 64, 72, 3, 3, 1, 1, 4),      # rows of more than one fragment
    (1, 14, 14, 128, 40, 3, 3, 2, 1, 4),
    (1, 5, 6, 64, 8, 3, 3, 1, 4, 4),        # padding wider than the filter
    (1, 7, 7, 512, 64, 3, 3, 1, 1, 4),      # depth over eight waves
    (1, 9, 8, 64, 24, 5, 5, 1, 2, 4),
    (1, 10, 9, 64, 16, 4, 7, 1, 3, 4),      # 28 taps
    (1, 9, 9, 64, 16, 6, 6, 1, 2, 4),       # 36 taps: more than a mask holds
    (1, 5, 3, 16, 4, 1, 1, 1, 0, 8),
    (1, 3, 11, 80, 20, 1, 1, 1, 0, 8),
    (1, 7, 7, 48, 20, 3, 3, 1, 1, 8),
    (2, 8, 8, 64, 36, 3, 3, 2, 1, 8),
    (3, 6, 7, 320, 160, 1, 1, 1, 0, 8),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_direct_layers(shape):
    import torch
    from paper_2202_06819_amd import qconv as q

    n, h, w, c, k, r, s, stride, pad, bits = shape
    dev = torch.device("cuda:0")
    g = np.random.default_rng([77, *shape])
    signed = bits == 8
    xr, wr = (qi.S8, qi.S8) if signed else (qi.U4, qi.S4)
    L = qi.Layer("direct", n, h, w, c, k, r, s, stride, pad, bits, signed, True, xr, wr)
    d = L.desc()
    x = g.integers(xr[0], xr[1] + 1, size=(n, c, h, w)).astype(np.int8)
    wt = g.integers(wr[0], wr[1] + 1, size=(k, c, r, s)).astype(np.int8)
    acc = oracle.qconv_layer(x, wt, bits=bits, x_signed=signed, w_signed=True, stride=(stride, stride), pad=(pad, pad),
                             threads=oracle_threads())["acc"].reshape(n, L.p, L.q, k)
    xp = q.pack(torch.from_numpy(x).to(dev), bits, signed)
    wp = q.pack(torch.from_numpy(wt).to(dev), bits, True)
    forms = epilogue_forms(g, k, bits, float(np.abs(acc).mean()), acc.shape)
    direct = 0
    for t in q.tiles():
        if t["variant"] != 2 or q.tile_status(d, t["id"]) != 0:
            continue
        prep = q.prepare_filters(d, wp, t["id"])
        announce(f"direct {shape} {t['name']} raw")
        y = q.conv2d(d, xp, prep, tile=t["id"], prepared=True)
        torch.cuda.synchronize()
        direct += q.last_kernel().startswith("direct_")
        assert_same(y.cpu().numpy(), acc.astype(np.int32), f"{shape} {t['name']} raw")
        for name, f in forms:
            if t["frag_p"] != 2 and "residual" not in name and name != "full range":
                continue   # the epilogue depends on the image's frag_k only
            announce(f"direct {shape} {t['name']} {name}")
            kw = dict(requant=True, mult=torch.from_numpy(f["mult"]).to(dev), shift=f["shift"], relu=False,
                      clamp=f["clamp"])
            if "bias" in f:
                kw["bias"] = torch.from_numpy(f["bias"]).to(dev)
            if "res" in f:
                packed = packed_values(f["res"], bits)
                kw.update(residual=torch.from_numpy(packed.view(np.int32) if bits == 4 else packed).to(dev),
                          residual_signed=f["res_signed"])
            y = q.conv2d(d, xp, prep, tile=t["id"], prepared=True, **kw)
            torch.cuda.synchronize()
            want = packed_values(requantised(acc, f["mult"].astype(np.int64), f["shift"], *f["clamp"], f.get("bias"),
                                  f.get("res")), bits)
            assert_same(y.cpu().numpy(), want, f"{shape} {t['name']} {name}")
    assert direct or r * s > 31, "no tile took the direct kernels"


def test_last_kernel_names_what_ran():
    """A direct launch names a direct kernel, whichever tile's image it reads; a
    schedule names its tile."""
    import torch
    from paper_2202_06819_amd import qconv as q

    dev = torch.device("cuda:0")
    L = qi.Layer("names", 1, 14, 14, 128, 64, 3, 3, 1, 1)
    d = L.desc()
    x = torch.zeros(q.layout(d)["x_bytes"], dtype=torch.uint8, device=dev)
    w = torch.zeros(q.layout(d)["w_bytes"], dtype=torch.uint8, device=dev)
    for t in q.tiles():
        if t["variant"] != 2 or q.tile_status(d, t["id"]) != 0:
            continue
        announce(f"last kernel, tile {t['name']}")
        prep = q.prepare_filters(d, w, t["id"])
        q.Conv2dCall(d, x, prep, schedule=dict(tile_id=t["id"]))()
        assert q.last_kernel() == t["name"] and q.last_launch()["threads"] == t["threads"]
        q.conv2d(d, x, prep, tile=t["id"], prepared=True)
        assert q.last_kernel().startswith(f"direct_b4_k{t['frag_k']}_"), q.last_kernel()
    torch.cuda.synchronize()


@pytest.mark.parametrize("n,h,w,c,k,stride,bits,tile", [
    (5, 83, 92, 1024, 24, 1, 8, "wide_b8_w4x1_f2x4_c64"),    # 58 us on its tile, 101 direct
    (28, 32, 41, 384, 24, 1, 8, "wide_b8_w4x1_f2x4_c64"),    # 23, 36
    (62, 63, 72, 128, 32, 2, 4, "wide_b4_w8x1_f1x4_c64"),    # 15, 26
])
def test_partial_blocks_are_priced(n, h, w, c, k, stride, bits, tile):
    """Few output channels from a 4-fragment image: the direct kernels compute
    the block's other channels too, so that these stay on their tile's kernel."""
    import torch
    from paper_2202_06819_amd import qconv as q

    dev = torch.device("cuda:0")
    d = qi.Layer("partial", n, h, w, c, k, 3, 3, stride, 1, bits, bits == 8, True).desc()
    x = torch.zeros(q.layout(d)["x_bytes"], dtype=torch.uint8, device=dev)
    tid = next(t["id"] for t in q.tiles() if t["name"] == tile)
    announce(f"partial blocks {n}x{h}x{w} {c}->{k} {tile}")
    q.conv2d(d, x, torch.zeros(q.prepared_filter_bytes(d, tid), dtype=torch.uint8, device=dev), tile=tid, prepared=True)
    torch.cuda.synchronize()
    assert q.last_kernel() == tile


def _full_splits(q, d, tile):
    """Split factors above one that leave no split empty."""
    chunks = q.max_splits(d, tile)
    return [s for s in range(2, chunks + 1) if -(-chunks // -(-chunks // s)) == s]


def test_a_split_is_run_as_asked():
    """`splits` > 1 launches tiles x splits workgroups of the wide tile, through
    a workspace, the no-alloc scratch and with a projection, on layers that
    run on direct kernels without a split."""
    import torch
    from paper_2202_06819_amd import qconv as q

    dev = torch.device("cuda:0")
    L = qi.Layer("split", 1, 14, 14, 256, 64, 3, 3, 2, 1)
    d = L.desc()
    x = torch.zeros(q.layout(d)["x_bytes"], dtype=torch.uint8, device=dev)
    w, w1 = (torch.zeros(q.layout(e)["w_bytes"], dtype=torch.uint8, device=dev) for e in (d, q.proj_desc(d)))
    for t in q.tiles():
        if t["variant"] != 2 or q.tile_status(d, t["id"]) != 0:
            continue
        tiles = -(-q.layout(d)["m"] // t["tile_p"]) * -(-L.k // t["tile_k"])
        prep = q.prepare_filters(d, w, t["id"])
        for splits in _full_splits(q, d, t["id"]):
            want = dict(grid=tiles * splits, threads=t["threads"])
            calls = {"workspace": q.Conv2dCall(d, x, prep, tile=t["id"], prepared=True, splits=splits),
                     "no-alloc": lambda: q.conv2d(d, x, prep, tile=t["id"], prepared=True, splits=splits, noalloc=True)}
            if q.proj_tile_status(d, t["id"]) == 0:
                calls["projection"] = q.ProjConv2dCall(d, x, q.prepare_filters_proj(d, w, w1, t["id"]), tile=t["id"],
                                                       splits=splits)
            for name, call in calls.items():
                announce(f"split {t['name']} {splits} {name}")
                call()
                launch = q.last_launch()
                assert {f: launch[f] for f in want} == want, (t["name"], splits, name, launch)
    torch.cuda.synchronize()


def test_direct_projection():
    """The strided 3x3 and its projection in one direct launch, against the two
    layers run apart by the wide kernels (a forced launch knob keeps them there)."""
    import torch
    from paper_2202_06819_amd import qconv as q

    dev = torch.device("cuda:0")
    for bits, n, h, c, k in ((4, 1, 14, 64, 72), (4, 2, 9, 256, 64), (8, 1, 11, 128, 36)):
        L = qi.Layer("proj", n, h, h, c, k, 3, 3, 2, 1, bits, bits == 8, True)
        d, dp = L.desc(), q.proj_desc(L.desc())
        g = np.random.default_rng([78, n, h, c, k])
        lo, hi = (0, 15) if bits == 4 else (-128, 127)
        x = q.pack(torch.from_numpy(g.integers(lo, hi + 1, size=(n, c, h, h)).astype(np.int8)).to(dev), bits, bits == 8)
        w3 = q.pack(torch.from_numpy(g.integers(-8, 8, size=(k, c, 3, 3)).astype(np.int8)).to(dev), bits, True)
        w1 = q.pack(torch.from_numpy(g.integers(-8, 8, size=(k, c, 1, 1)).astype(np.int8)).to(dev), bits, True)
        m3, m1 = (torch.from_numpy(g.integers(1 << 14, 1 << 15, size=k).astype(np.int32)).to(dev) for _ in range(2))
        b1 = torch.from_numpy(g.integers(-200, 200, size=k).astype(np.int32)).to(dev)
        direct = 0
        for t in q.tiles():
            if q.proj_tile_status(d, t["id"]) != 0 or q.tile_status(dp, t["id"]) != 0:
                continue
            announce(f"direct projection {bits} {n} {h} {c} {k} {t['name']}")
            y, yp = q.ProjConv2dCall(d, x, q.prepare_filters_proj(d, w3, w1, t["id"]), tile=t["id"], requant=True,
                                     mult=m3, shift=22, relu=False, clamp=(lo, hi),
                                     proj=dict(mult=m1, shift=20, relu=False, clamp=(lo, hi), bias=b1))()
            direct += q.last_kernel().startswith("direct_")
            sch = dict(tile_id=t["id"], wg_per_cu=1)
            w = [q.Conv2dCall(d, x, q.prepare_filters(d, w3, t["id"]), requant=True, mult=m3, shift=22, relu=False,
                              clamp=(lo, hi), schedule=sch)(),
                 q.Conv2dCall(dp, x, q.prepare_filters(dp, w1, t["id"]), requant=True, mult=m1, shift=20, relu=False,
                              clamp=(lo, hi), bias=b1, schedule=sch)()]
            torch.cuda.synchronize()
            assert_same(y.cpu().numpy(), w[0].cpu().numpy(), f"projection {t['name']} layer")
            assert_same(yp.cpu().numpy(), w[1].cpu().numpy(), f"projection {t['name']} projection")
        assert direct, f"no tile took the direct kernels for {n}x{h}x{h} {c}->{k}"
