"""Every form of the direct kernels (wave tile, depth, steps in flight, filters
resident or not, two steps a load, one or several rounds), named instead of
chosen, on small layers at the edges of its tiles and with every epilogue,
against the oracle's sums; and the same layers on the tile's own kernel."""
import re

import numpy as np
import pytest

import oracle
import qconv_inputs as qi
from _util import announce, assert_same, epilogue_forms, oracle_threads, packed_values, requantised

pytestmark = pytest.mark.gpu

# (n, h, w, c, k, r, s, stride, pad_h, pad_w), c for 4-bit operands (8-bit: half of
# a 32, else the same).  Pixels that are no multiple of any wave tile, channels
# that fill no pair or block, and for each kind of filter one to several rounds
# of the steps a form has in flight.
SHAPES = [
    (1, 5, 7, 32, 24, 1, 1, 1, 0, 0),         # half a step
    (2, 3, 11, 64, 72, 1, 1, 1, 0, 0),        # one step
    (1, 9, 13, 96, 40, 1, 1, 1, 0, 0),        # a step and a half: the last load ends at the tensor's end
    (1, 6, 11, 128, 136, 1, 1, 1, 0, 0),      # two steps, whole pairs
    (3, 7, 9, 256, 72, 1, 1, 1, 0, 0),        # four
    (1, 5, 13, 512, 40, 1, 1, 1, 0, 0),       # eight
    (1, 4, 9, 1088, 72, 1, 1, 1, 0, 0),       # seventeen: rounds with a remainder
    (1, 5, 9, 1664, 40, 1, 1, 1, 0, 0),       # twenty-six, whole pairs
    (3, 37, 41, 32, 2056, 1, 1, 1, 0, 0),     # more pixel tiles than a resident launch's waves
    (3, 37, 41, 128, 2056, 1, 1, 1, 0, 0),
    (2, 9, 11, 32, 24, 3, 3, 1, 1, 1),        # half a step a tap
    (1, 7, 18, 64, 72, 3, 3, 1, 1, 1),        # rows of more than a fragment
    (2, 11, 9, 128, 40, 3, 3, 2, 1, 1),
    (1, 8, 7, 192, 136, 3, 3, 1, 1, 1),       # three rounds of nine
    (1, 6, 5, 64, 24, 5, 5, 1, 4, 4),         # padding wider than the filter's half
    (2, 13, 9, 64, 40, 4, 1, 1, 0, 0),        # a column of taps
    (2, 9, 9, 256, 24, 1, 1, 2, 0, 0),        # strided 1x1
    (2, 33, 31, 64, 1032, 2, 2, 1, 0, 1),     # more pixel tiles than a resident launch's waves
]
# images of 2- and 4-fragment blocks, of one and several blocks a channel tile, of 64- and 128-channel chunks
TILES = {4: ("wide_b4_w4x2_f2x2_c64", "wide_b4_w4x1_f2x4_c64", "wide_b4_w2x4_f4x4_c64", "wide_b4_w4x2_f2x2_c128",
             "wide_b4_w2x2_f4x4_c128"),
         8: ("wide_b8_w4x2_f2x2_c64", "wide_b8_w4x1_f2x4_c64", "wide_b8_w1x4_f4x4_c64")}

# what the forms are made of: (fragments x pairs, steps in flight, kind), and which of one round and several there is
DEPTH = {("f1x1", 9, ""): "both", ("f2x1", 3, ""): "several", ("f2x2", 3, ""): "several",
         ("f1x1", 4, "_1x1"): "one", ("f2x1", 4, "_1x1"): "one", ("f1x1", 8, "_1x1"): "both",
         ("f2x1", 8, "_1x1"): "both", ("f2x2", 4, "_1x1"): "both", ("f4x2", 4, "_1x1"): "both"}
RESIDENT = {("f2x2", 3, ""): "several", ("f2x2", 1, "_1x1"): "one", ("f4x2", 1, "_1x1"): "one",
            ("f2x2", 2, "_1x1"): "one", ("f4x2", 2, "_1x1"): "one", ("f2x2", 4, "_1x1"): "both"}
TWO = {("f2x2", 2, "_1x1_two"): "one", ("f4x2", 2, "_1x1_two"): "one", ("f2x2", 4, "_1x1_two"): "both"}


def _expected(bits):
    out = set()
    for kind, table in (("depth", DEPTH), ("resident", RESIDENT), ("resident", TWO if bits == 4 else {})):
        for (tile, la, mid), rounds in table.items():
            for k in (2, 4):
                for ext in ("", "_ext"):
                    if rounds != "several":
                        out.add((k, tile, la, kind + mid + ext))
                    if rounds != "one":
                        out.add((k, tile, la, kind + mid + "_rounds" + ext))
    return out


def _instance(name):
    m = re.fullmatch(r"direct_b\d_k(\d)_(f\dx\d)_d\d_t\d_l(\d)_(\w+)", name)
    assert m, name
    return int(m[1]), m[2], int(m[3]), m[4]


def _case(shape, bits):
    n, h, w, c, k, r, s, stride, ph, pw = shape
    if bits == 8 and c == 32:
        c = 16
    g = np.random.default_rng([79, bits, *shape])
    signed = bits == 8
    lo, hi = (-128, 127) if signed else (0, 15)
    x = g.integers(lo, hi + 1, size=(n, c, h, w)).astype(np.int8)
    wt = g.integers(*((-128, 128) if signed else (-8, 8)), size=(k, c, r, s)).astype(np.int8)
    d = dict(n=n, h=h, w=w, c=c, k=k, r=r, s=s, stride_h=stride, stride_w=stride, pad_h=ph, pad_w=pw, bits=bits,
             x_signed=int(signed), w_signed=1)
    acc = oracle.qconv_layer(x, wt, bits=bits, x_signed=signed, w_signed=True, stride=(stride, stride), pad=(ph, pw),
                             threads=oracle_threads())["acc"]
    return g, d, x, wt, acc


def _args(f, bits, dev):
    import torch
    kw = dict(requant=True, mult=torch.from_numpy(f["mult"]).to(dev), shift=f["shift"], relu=False, clamp=f["clamp"])
    if "bias" in f:
        kw["bias"] = torch.from_numpy(f["bias"]).to(dev)
    if "res" in f:
        packed = packed_values(f["res"], bits)
        kw.update(residual=torch.from_numpy(packed.view(np.int32) if bits == 4 else packed).to(dev),
                  residual_signed=f["res_signed"])
    return kw


@pytest.mark.parametrize("bits", [4, 8])
def test_every_form_and_epilogue(bits):
    import torch
    from paper_2202_06819_amd import qconv as q

    dev = torch.device("cuda:0")
    ids = {t["name"]: t["id"] for t in q.tiles()}
    reached, ran = set(), set()
    for shape in SHAPES:
        g, d, x, wt, acc = _case(shape, bits)
        xp = q.pack(torch.from_numpy(x).to(dev), bits, bits == 8)
        wp = q.pack(torch.from_numpy(wt).to(dev), bits, True)
        wants, kws = {"raw": acc.astype(np.int32)}, {"raw": {}}
        for name, f in epilogue_forms(g, d["k"], bits, float(np.abs(acc).mean()), acc.shape):
            wants[name] = packed_values(requantised(acc, f["mult"].astype(np.int64), f["shift"], *f["clamp"], f.get("bias"),
                                         f.get("res")), bits)
            kws[name] = _args(f, bits, dev)
        want = {name: torch.from_numpy(np.ascontiguousarray(v).view(np.int32 if v.dtype != np.int8 else np.int8)).to(dev)
                for name, v in wants.items()}
        for tile in TILES[bits]:
            if q.tile_status(d, ids[tile]) != 0:
                continue
            prep = q.prepare_filters(d, wp, ids[tile])
            for form in range(-1, q.form_count()):
                announce(f"form {form} {bits}-bit {shape} {tile}")
                for name, kw in kws.items():
                    call = q.Conv2dCall(d, xp, prep, tile=ids[tile], prepared=True, form=form, **kw)
                    try:
                        y = call()
                    except q.QConvError as e:
                        assert e.status == q.EUNSUPPORTED and form >= 0, e
                        break
                    kernel = q.last_kernel()
                    if form < 0:
                        assert kernel == tile
                    else:
                        reached.add(_instance(kernel))
                        ran.add(form)
                        assert kernel.endswith("_ext") == ("bias" in kw or "residual" in kw), (name, kernel)
                    if not torch.equal(y.view(want[name].dtype), want[name]):
                        assert_same(y.cpu().numpy(), wants[name], f"form {form} ({kernel}) {shape} {tile} {name}")
    assert ran == set(range(q.form_count())) - ({24, 25, 27, 28} if bits == 8 else set())   # (two steps a load: 4 bits)
    assert reached == _expected(bits), (sorted(_expected(bits) - reached), sorted(reached - _expected(bits)))


@pytest.mark.parametrize("bits", [4, 8])
def test_every_form_of_a_projection(bits):
    """The 3x3 layer and its projection in one launch: the tile's kernel, and
    every direct form that takes one, raw and requantised with a bias."""
    import torch
    from paper_2202_06819_amd import qconv as q

    dev = torch.device("cuda:0")
    ran = set()
    for n, h, w, c, k, stride in ((1, 9, 11, 32, 40, 2), (2, 7, 18, 64, 72, 1), (1, 14, 13, 192, 40, 2), (1, 7, 7, 512, 136, 2)):
        g, d, x, w3, acc = _case((n, h, w, c, k, 3, 3, stride, 1, 1), bits)
        w1 = g.integers(*((-128, 128) if bits == 8 else (-8, 8)), size=(k, d["c"], 1, 1)).astype(np.int8)
        acc1 = oracle.qconv_layer(x, w1, bits=bits, x_signed=bits == 8, w_signed=True, stride=(stride, stride),
                                  pad=(0, 0), threads=oracle_threads())["acc"]
        xp = q.pack(torch.from_numpy(x).to(dev), bits, bits == 8)
        p3, p1 = (q.pack(torch.from_numpy(f).to(dev), bits, True) for f in (w3, w1))
        f3, f1 = (dict(epilogue_forms(g, k, bits, float(np.abs(a).mean()), a.shape))["bias"] for a in (acc, acc1))
        k3, k1 = _args(f3, bits, dev), _args(f1, bits, dev)
        k1.pop("requant")
        wants = [(acc.astype(np.int32), acc1.astype(np.int32))]
        wants.append(tuple(packed_values(requantised(a, f["mult"].astype(np.int64), f["shift"], *f["clamp"], f["bias"]), bits)
                           for a, f in ((acc, f3), (acc1, f1))))
        for t in q.tiles():
            if q.proj_tile_status(d, t["id"]) != 0:
                continue
            prep = q.prepare_filters_proj(d, p3, p1, t["id"])
            for form in range(-1, q.form_count()):
                announce(f"projection form {form} {bits}-bit {n}x{h}x{w} {c}->{k} {t['name']}")
                for kw, want in zip(({}, dict(k3, proj=k1)), wants):
                    try:
                        got = q.ProjConv2dCall(d, xp, prep, tile=t["id"], form=form, **kw)()
                    except q.QConvError as e:
                        assert e.status == q.EUNSUPPORTED and form >= 0, e
                        break
                    assert q.last_kernel().startswith("direct_") == (form >= 0)
                    ran.add(form)
                    for y, v, what in zip(got, want, ("layer", "projection")):
                        assert_same(y.cpu().numpy(), v, f"form {form} {t['name']} {what}")
    assert ran == set(range(-1, 9))   # the depth forms of filters larger than 1x1
