"""Plain reads of frames whose rows are not whole 4-pixel units or not dword
aligned, contiguous (one row of units) and cropped, into outputs at every
element alignment: the oracle's bits, and nothing written outside them."""
import numpy as np
import pytest
import torch

import datagen
import fkhelpers as H
import oracle
import paper_2508_07071_amd as fk

pytestmark = pytest.mark.gpu
PAD = 64  # canary elements on both sides of an output


@pytest.mark.parametrize("din", ["u8", "f16", "f32"])
@pytest.mark.parametrize("dout", ["f16", "f32"])
@pytest.mark.parametrize("layout", ["packed", "planar"])
@pytest.mark.parametrize("c", [1, 3, 4])
def test_ragged_frames(din, dout, layout, c):
    g = datagen.rng(c)
    ops = [{"kind": "cvt", "k": []}, {"kind": "sub", "k": [100.0]}, {"kind": "div", "k": [0.75]}]
    ch = {"read": {"kind": "plain", "dtype": din, "channels": c, "out_w": 0, "out_h": 0}, "ops": ops,
          "write": {"dtype": dout, "layout": layout}}
    sizes = [(1, 1), (2, 3), (3, 2), (5, 7), (4, 4), (255, 3), (257, 5), (1023, 2), (1025, 9), (63, 65)]
    frames = [datagen.frame(g, h, w, c, din) for w, h in sizes]
    items = [{"frame": i, "x": 0, "y": 0, "w": w, "h": h} for i, (w, h) in enumerate(sizes)]       # whole
    items += [{"frame": i, "x": 0, "y": 1, "w": w, "h": h - 1} for i, (w, h) in enumerate(sizes) if h > 1]
    items += [{"frame": i, "x": x, "y": 0, "w": w - x - 1, "h": h} for i, (w, h) in enumerate(sizes)
              for x in (1, 2, 3) if w > x + 1]                                                    # cropped
    refs = oracle.run_chain(ch, frames, items)
    dev = H.to_dev(frames)
    dt = fk.TORCH_DTYPE[dout]
    for cfg in ((64, 1), (256, 2), (128, 8)):
        bufs, outs = [], []
        for j, it in enumerate(items):
            n = it["w"] * it["h"] * c
            off = PAD + j % 5  # every alignment of the first element
            b = torch.full((n + 2 * PAD + 8,), 7.5, dtype=dt, device="cuda")
            bufs.append((b, off, n))
            outs.append(b[off:off + n])
        with H.Plan(ch, len(items), strict=True, tier=1) as p:
            p.set_config(*cfg)
            p.run(dev, items, outs=outs)
        for j, ((b, off, n), r) in enumerate(zip(bufs, refs)):
            h = b.cpu().numpy()
            H.assert_bitexact(h[off:off + n].reshape(r["out"].shape), r["out"], f"{cfg} item {j} {items[j]}")
            assert (h[:off] == 7.5).all() and (h[off + n:] == 7.5).all(), (cfg, items[j])


def test_ragged_compile_time_chain_and_graph():
    """The same frames through a compile-time chain, eager and graph replay."""
    g = datagen.rng(9)
    ch = datagen.muladd_chain(4, g)
    sizes = [(1, 1), (7, 3), (255, 3), (1025, 9), (640, 4)]
    frames = [datagen.frame(g, h, w, 3) for w, h in sizes]
    items = [{"frame": i, "x": 0, "y": 0, "w": w, "h": h} for i, (w, h) in enumerate(sizes)]
    refs = oracle.run_chain(ch, frames, items)
    dev = H.to_dev(frames)
    for graph in (False, True):
        with H.Plan(ch, len(items), strict=True, use_graph=graph) as p:
            for _ in range(3):
                got = H.host(p.run(dev, items))
                for a, r in zip(got, refs):
                    H.assert_bitexact(a, r["out"], f"graph {graph}")


@pytest.mark.parametrize("w,h,layout", [(61, 5, "packed"), (61, 7, "planar"), (63, 1, "packed"), (257, 3, "planar"),
                                        (64, 4, "packed")])
def test_strips_of_one_frame(w, h, layout):
    """More whole-row strips of one frame than the full kernel-argument form
    holds, outputs at a constant stride."""
    g = datagen.rng(w)
    n, c = 45, 3
    ch = {"read": {"kind": "plain", "dtype": "u8", "channels": c, "out_w": 0, "out_h": 0},
          "ops": [{"kind": "mul", "k": [0.5]}, {"kind": "div", "k": [3.0]}],
          "write": {"dtype": "f32", "layout": layout}}
    fr = datagen.frame(g, n * h, w, c)
    items = [{"frame": 0, "x": 0, "y": i * h, "w": w, "h": h} for i in range(n)]
    refs = oracle.run_chain(ch, [fr], items)
    out = torch.full((n,) + tuple(fk.out_shape(ch, items[0])), float("nan"), device="cuda")
    for cfg in ((64, 1), (256, 1), (128, 8)):
        out.fill_(float("nan"))
        with H.Plan(ch, n, strict=True, tier=1) as p:
            p.set_config(*cfg)
            p.run(H.to_dev([fr]), items, outs=[out[i] for i in range(n)])
        got = out.cpu().numpy()
        for i, r in enumerate(refs):
            H.assert_bitexact(got[i], r["out"], f"{cfg} strip {i}")
