"""Bilinear reads on launches large enough for pixel-strided lanes, every
element type, channel count, output type and layout: ROIs of one and two
columns, at every frame edge, enlarged and reduced, against the oracle bit for
bit; and the same items on a small launch (4-pixel units)."""
import numpy as np
import pytest
import torch

import datagen
import fkhelpers as H
import oracle
import paper_2508_07071_amd as fk

pytestmark = pytest.mark.gpu


def items_of(fw, fh, big):
    rois = [(0, 0, fw, fh), (fw - 1, 0, 1, fh), (fw - 2, fh - 1, 2, 1), (0, fh - 1, fw, 1), (3, 2, 2, fh - 2),
            (fw - 31, fh - 17, 31, 17), (1, 1, 5, 3)]
    sizes = [(512, 512), (517, 509), (511, 513), (640, 400), (333, 800), (700, 377), (64, 65)] if big else \
            [(9, 5), (4, 4), (1, 1), (3, 17), (33, 2), (65, 6), (2, 3)]
    return [{"frame": i % 2, "x": x, "y": y, "w": w, "h": h, "out_w": ow, "out_h": oh}
            for i, ((x, y, w, h), (ow, oh)) in enumerate(zip(rois, sizes))]


@pytest.mark.parametrize("din", ["u8", "f16", "f32"])
@pytest.mark.parametrize("c", [1, 3, 4])
@pytest.mark.parametrize("dout,layout", [("f32", "packed"), ("f16", "packed"), ("f32", "planar"), ("f16", "planar")])
def test_strided_gathers(din, c, dout, layout):
    g = datagen.rng(7 * c)
    fw, fh = 61, 37
    frames = [datagen.frame(g, fh, fw, c, din) for _ in range(2)]
    ch = {"read": {"kind": "crop_resize", "dtype": din, "channels": c, "out_w": 0, "out_h": 0},
          "ops": [{"kind": "swap", "k": []}, {"kind": "sub", "k": [100.0]}, {"kind": "div", "k": [0.75]}],
          "write": {"dtype": dout, "layout": layout}}
    dev = H.to_dev(frames)
    dt = fk.TORCH_DTYPE[dout]
    for big in (True, False):
        items = items_of(fw, fh, big)
        assert not big or sum(it["out_w"] * it["out_h"] for it in items) >= 1 << 20
        refs = oracle.run_chain(ch, frames, items)
        for cfg in ((256, 1), (64, 4)):
            bufs = []
            for i, it in enumerate(items):  # canaries around each output, its start at every element alignment
                n = it["out_w"] * it["out_h"] * c
                bufs.append((torch.full((n + 80,), 7.5, dtype=dt, device="cuda"), 32 + i % 5, n))
            with H.Plan(ch, len(items), strict=True) as p:
                p.set_config(*cfg)
                p.run(dev, items, outs=[b[o:o + n] for b, o, n in bufs])
            for i, ((b, o, n), r) in enumerate(zip(bufs, refs)):
                h = b.cpu().numpy()
                H.assert_bitexact(h[o:o + n].reshape(r["out"].shape), r["out"], f"{cfg} big={big} item {i}")
                assert (h[:o] == 7.5).all() and (h[o + n:] == 7.5).all(), (cfg, big, i)
