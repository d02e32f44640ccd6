"""Batches whose items travel in the kernel arguments, around the capacity of
each form: corners of one frame (1:1 reads, 624 a launch), ROIs of one frame
(312), several frames of one geometry (156, two launches, then the table).
The oracle's bits, with unequal frames and ROIs at every byte alignment."""
import numpy as np
import pytest
import torch

import datagen
import fkhelpers as H
import oracle
import paper_2508_07071_amd as fk

pytestmark = pytest.mark.gpu

CHAINS = {
    "plain": ({"kind": "plain", "dtype": "u8", "channels": 3}, {"dtype": "f32", "layout": "planar"}),
    "resize": ({"kind": "crop_resize", "dtype": "u8", "channels": 3}, {"dtype": "f32", "layout": "planar"}),
    "nearest": ({"kind": "crop_nearest", "dtype": "f16", "channels": 1}, {"dtype": "f16", "layout": "packed"}),
    "nv12": ({"kind": "nv12", "dtype": "u8", "channels": 3}, {"dtype": "f32", "layout": "packed"}),
    "double": ({"kind": "plain", "dtype": "f32", "channels": 1}, {"dtype": "f64", "layout": "packed"}),
    "stats": ({"kind": "plain", "dtype": "u8", "channels": 4}, {"dtype": "f64", "layout": "stats"}),
    "loop": ({"kind": "plain", "dtype": "u8", "channels": 1}, {"dtype": "f32", "layout": "packed"}),
}


def case(kind, n, frames):
    g = datagen.rng(n + frames)
    read, write = CHAINS[kind]
    fh, fw = 40, 62
    ch = {"read": dict(read, out_w=0, out_h=0), "write": write,
          "ops": [{"kind": "cvt", "k": []}, {"kind": "sub", "k": [100.0]}, {"kind": "div", "k": [0.7]}]}
    if kind == "loop":
        ch["ops"] = [{"kind": "mul", "k": [0.75]}, {"kind": "add", "k": [0.5]}, {"kind": "loop", "span": 2, "count": 40}]
    frs = [datagen.nv12_frame(g, fh, fw) if kind == "nv12" else datagen.frame(g, fh, fw, read["channels"], read["dtype"])
           for _ in range(frames)]
    resizing = kind in ("resize", "nearest")
    items = []
    for b in range(n):
        w, h = (int(g.integers(1, 30)), int(g.integers(1, 20))) if resizing else (13, 6)
        items.append({"frame": b % frames, "x": int(g.integers(0, fw - w + 1)), "y": int(g.integers(0, fh - h + 1)),
                      "w": w, "h": h, "out_w": 9 if resizing else w, "out_h": 5 if resizing else h})
    return ch, frs, items


@pytest.mark.parametrize("kind", list(CHAINS))
@pytest.mark.parametrize("n,frames", [(33, 1), (312, 1), (313, 1), (624, 1), (625, 1), (33, 3), (156, 5), (157, 5),
                                      (312, 7), (313, 7)])
def test_forms(kind, n, frames):
    ch, frs, items = case(kind, n, frames)
    refs = oracle.run_chain(ch, frs, items)
    dt = fk.TORCH_DTYPE[ch["write"]["dtype"]]
    out = torch.full((n,) + tuple(fk.out_shape(ch, items[0])), float("nan"), dtype=dt, device="cuda")
    with H.Plan(ch, n, strict=True) as p:
        p.run(H.to_dev(frs), items, outs=[out[i] for i in range(n)])
    got = out.cpu().numpy()
    for i, r in enumerate(refs):
        if kind == "stats":  # min and max exact, sums of 78 values of 32 bits within 78 roundings of 2^-53
            H.assert_bitexact(got[i][:, :2], r["out"][:, :2], f"item {i}")
            np.testing.assert_allclose(got[i][:, 2:], r["out"][:, 2:], rtol=1e-12, atol=1e-9)
        else:
            H.assert_bitexact(got[i], r["out"], f"item {i} of {n} ({frames} frames)")
