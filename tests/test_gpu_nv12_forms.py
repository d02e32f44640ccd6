"""Batches whose items travel in the kernel arguments, NV12 above all, on frames whose
base and pitch are multiples of 4: a 1:1 read then takes whole dwords at the
columns that are multiples of 4 and bytes at the others, item by item, also
where the last launch of a split batch holds one item (625 and 1249 corners
of one frame, 157 and 313 ROIs).  The oracle's bits."""
import pytest
import torch

import datagen
import fkhelpers as H
import oracle
import paper_2508_07071_amd as fk

pytestmark = pytest.mark.gpu

FH, FW = 40, 64


def batch(kind, n, frames, last_x):
    g = datagen.rng(7 * n + 3 * frames + last_x)
    ch = {"read": {"kind": kind, "dtype": "u8", "channels": 3, "out_w": 0, "out_h": 0},
          "ops": [{"kind": "cvt", "k": []}, {"kind": "sub", "k": [100.0]}, {"kind": "div", "k": [0.7]}],
          "write": {"dtype": "f32", "layout": "planar"}}
    frs = [datagen.nv12_frame(g, FH, FW) for _ in range(frames)]
    items = []
    for b in range(n):
        w, h = (13, 6) if kind == "nv12" else (int(g.integers(1, 30)), int(g.integers(1, 20)))
        x = last_x if b == n - 1 else int(g.integers(0, FW - w + 1))
        items.append({"frame": b % frames, "x": x, "y": int(g.integers(0, FH - h + 1)), "w": w, "h": h,
                      "out_w": w if kind == "nv12" else 9, "out_h": h if kind == "nv12" else 5})
    return ch, frs, items


def check(ch, items, frs, dframes):
    refs = oracle.run_chain(ch, frs, items)
    n = len(items)
    dt = fk.TORCH_DTYPE[ch["write"]["dtype"]]
    out = torch.full((n,) + tuple(fk.out_shape(ch, items[0])), float("nan"), dtype=dt, device="cuda")
    with H.Plan(ch, n, strict=True) as p:
        p.run(dframes, items, outs=[out[i] for i in range(n)])
    got = out.cpu().numpy()
    for i, r in enumerate(refs):
        H.assert_bitexact(got[i], r["out"], f"item {i} of {n}, x = {items[i]['x']}")


@pytest.mark.parametrize("last_x", [0, 1, 2, 3])
@pytest.mark.parametrize("kind,n,frames", [("nv12", 1, 1), ("nv12", 33, 1), ("nv12", 624, 1), ("nv12", 625, 1),
                                           ("nv12", 1249, 1), ("nv12", 33, 5), ("nv12", 156, 5), ("nv12", 157, 5),
                                           ("nv12_resize", 313, 1), ("nv12_resize", 157, 5)])
def test_columns(kind, n, frames, last_x):
    ch, frs, items = batch(kind, n, frames, last_x)
    check(ch, items, frs, H.to_dev(frs))


@pytest.mark.parametrize("n", [33, 157])
@pytest.mark.parametrize("odd_frame", [0, 2])
@pytest.mark.parametrize("offset", [1, 2])
def test_frames_of_mixed_alignment(n, odd_frame, offset):
    """Several frames of one geometry, one of them at an unaligned base."""
    ch, frs, items = batch("nv12", n, 3, 1)
    dframes = H.to_dev(frs)
    size = frs[odd_frame].size
    buf = torch.zeros(size + 16, dtype=torch.uint8, device="cuda")
    buf[offset:offset + size] = dframes[odd_frame].reshape(-1)
    dframes[odd_frame] = buf[offset:offset + size].view(frs[odd_frame].shape)
    check(ch, items, frs, dframes)


@pytest.mark.parametrize("kind", ["crop_resize", "nv12_resize"])
@pytest.mark.parametrize("dtype,layout", [("f32", "planar"), ("f16", "packed")])
@pytest.mark.parametrize("n,frames", [(157, 5), (313, 1)])
def test_split_run_in_strided_lanes(kind, dtype, layout, n, frames):
    """A run of 2^20 pixels and more takes pixel-strided lanes in each of its
    launches, the last one of a single item (NV12 and BGR)."""
    ch, frs, items = batch("nv12_resize", n, frames, 3)
    if kind == "crop_resize":
        g = datagen.rng(n)
        frs = [datagen.frame(g, FH, FW, 3, "u8") for _ in range(frames)]
    ch["read"]["kind"], ch["write"] = kind, {"dtype": dtype, "layout": layout}
    for it in items:
        it.update(out_w=97, out_h=71)
    assert n * 97 * 71 >= 1 << 20
    check(ch, items, frs, H.to_dev(frs))
