"""Items much smaller than the launch's tiles: waves, and register groups of a
wave, that hold no pixel of the item, next to waves with a few.  Every read,
write and element type at the widest tiles, outputs at line-aligned and
unaligned starts with canaries around them, against the oracle bit for bit
(stats: min and max bit for bit, sums of at most 600 values within 600
roundings of 2^-53)."""
import numpy as np
import pytest
import torch

import datagen
import fkhelpers as H
import oracle
import paper_2508_07071_amd as fk

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (3, 1), (4, 1), (5, 2), (13, 7), (64, 4), (257, 1), (1, 66), (9, 65)]
READS = [("plain", "u8", 3), ("plain", "f16", 1), ("plain", "f32", 4), ("crop_resize", "u8", 1), ("crop_resize", "u8", 4),
         ("crop_resize", "f16", 3), ("crop_resize", "f32", 4), ("crop_nearest", "u8", 4), ("crop_nearest", "f32", 1),
         ("nv12", "u8", 3), ("nv12_resize", "u8", 3)]


def case(kind, dtype, c, write):
    g = datagen.rng(c + len(kind))
    fh, fw = 72, 262
    ch = {"read": {"kind": kind, "dtype": dtype, "channels": c, "out_w": 0, "out_h": 0}, "write": write,
          "ops": [{"kind": "sub", "k": [100.0]}, {"kind": "div", "k": [0.7]}]}
    frs = [datagen.nv12_frame(g, fh, fw) if kind.startswith("nv12") else datagen.frame(g, fh, fw, c, dtype)]
    items = []
    for ow, oh in SIZES:
        w, h = (ow, oh) if kind in ("plain", "nv12") else (int(g.integers(1, fw + 1)), int(g.integers(1, fh + 1)))
        items.append({"frame": 0, "x": int(g.integers(0, fw - w + 1)), "y": int(g.integers(0, fh - h + 1)), "w": w,
                      "h": h, "out_w": ow, "out_h": oh})
    return ch, frs, items


def run(ch, frs, items, cfg):
    refs = oracle.run_chain(ch, frs, items)
    dt = fk.TORCH_DTYPE[ch["write"]["dtype"]]
    lead = 64 if dt == torch.float16 else 32  # to the next 128-byte line; the next four starts are unaligned
    bufs = []
    for i, it in enumerate(items):
        n = int(np.prod(fk.out_shape(ch, it)))
        bufs.append((torch.full((n + 80,), 7.5, dtype=dt, device="cuda"), lead + i % 5, n))
    with H.Plan(ch, len(items), strict=True) as p:
        p.set_config(*cfg)
        p.run(H.to_dev(frs), items, outs=[b[o:o + n].view(fk.out_shape(ch, it)) for (b, o, n), it in zip(bufs, items)])
    for i, ((b, o, n), r) in enumerate(zip(bufs, refs)):
        h = b.cpu().numpy()
        got = h[o:o + n].reshape(r["out"].shape)
        if ch["write"]["layout"] == "stats":
            H.assert_bitexact(got[:, :2], r["out"][:, :2], f"{cfg} item {i}")
            np.testing.assert_allclose(got[:, 2:], r["out"][:, 2:], rtol=1e-12, atol=1e-9)
        else:
            H.assert_bitexact(got, r["out"], f"{cfg} item {i}")
        assert (h[:o] == 7.5).all() and (h[o + n:] == 7.5).all(), (cfg, i)


@pytest.mark.parametrize("cfg", [(1024, 8), (512, 2), (64, 8)])
@pytest.mark.parametrize("read", READS, ids=lambda r: "-".join(map(str, r)))
def test_small_items_in_wide_tiles(read, cfg):
    for write in ({"dtype": "f32", "layout": "planar"}, {"dtype": "f16", "layout": "packed"},
                  {"dtype": "f32", "layout": "packed"}, {"dtype": "f64", "layout": "stats"}):
        run(*case(*read, write), cfg)


@pytest.mark.parametrize("cfg", [(1024, 8), (256, 1), (64, 8)])
@pytest.mark.parametrize("dtype", ["u8", "f16", "f32", "f64"])
@pytest.mark.parametrize("c", [1, 3, 4])
def test_small_fp64_items(dtype, c, cfg):
    for layout in ("planar", "packed"):
        run(*case("plain", dtype, c, {"dtype": "f64", "layout": layout}), cfg)
