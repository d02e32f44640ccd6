"""Stats of items that are not whole 4-pixel units or not dword aligned: whole
frames of odd width, strips and crops, in the integer path (u8, cast only) and
the float path, at the smallest and largest tiles."""
import pytest

import datagen
from fkhelpers import to_dev
from test_gpu_stats import check, oracle_refs, run_stats

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("din,ops", [("u8", False), ("u8", True), ("f16", False), ("f32", True)])
@pytest.mark.parametrize("c", [1, 3, 4])
def test_ragged_items(din, ops, c):
    g = datagen.rng(c)
    chain = {"read": {"kind": "plain", "dtype": din, "channels": c, "out_w": 0, "out_h": 0},
             "ops": [{"kind": "swap", "k": []}, {"kind": "cvt", "k": []}] +
                    ([{"kind": "sub", "k": [100.0]}, {"kind": "div", "k": [0.75]}] if ops else [])}
    sizes = [(1, 1), (2, 3), (3, 70), (5, 7), (4, 4), (101, 37), (1023, 5), (257, 300)]
    frames = [datagen.frame(g, h, w, c, din) for w, h in sizes]
    items = [{"frame": i, "x": 0, "y": 0, "w": w, "h": h} for i, (w, h) in enumerate(sizes)]
    items += [{"frame": i, "x": 0, "y": 1, "w": w, "h": h - 1} for i, (w, h) in enumerate(sizes) if h > 1]
    items += [{"frame": i, "x": x, "y": 0, "w": w - x - 1, "h": h} for i, (w, h) in enumerate(sizes)
              for x in (1, 2, 3) if w > x + 1]
    st, ims = oracle_refs(chain, frames, items)
    dev = to_dev(frames)
    for cfg in ((256, 8), (64, 1), (1024, 4)):
        got = run_stats(chain, dev, items, strict=True, config_source=1, manual=cfg)
        for i, it in enumerate(items):
            check(got[i], st[i], ims[i], True, f"{din} x{c} {cfg} {it}")
