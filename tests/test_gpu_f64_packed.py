"""Packed fp64 writes at the sizes where a wave stores its pixels as one run
(all 64 lanes hold a pixel) and where it stores lane by lane: pixel counts
around a wave and a block, 3 and 4 channels, outputs that are 8- but not
16-byte aligned.  The values are the planar plan's, bit for bit, and nothing
is written before or after the output."""
import numpy as np
import pytest
import torch

import datagen
from fkhelpers import Plan, host, to_dev

pytestmark = pytest.mark.gpu


def chain(C, layout):
    return {"read": {"kind": "plain", "dtype": "u8", "channels": C, "out_w": 0, "out_h": 0},
            "ops": [{"kind": "cvt", "k": []}, {"kind": "mul", "k": [datagen.f32(1 / 255)]},
                    {"kind": "sub", "k": [datagen.f32(0.1 * c) for c in range(C)]}],
            "write": {"dtype": "f64", "layout": layout}}


@pytest.mark.parametrize("C", [3, 4])
@pytest.mark.parametrize("w,h", [(1, 1), (63, 1), (64, 1), (13, 5), (128, 1), (43, 3), (257, 5)])
def test_packed_runs_match_planar(C, w, h):
    print("[case] packed fp64, C", C, "pixels", w, "x", h, flush=True)
    frame = datagen.frame(datagen.rng(w * h + C), h + 2, w + 3, C)
    items = [{"frame": 0, "x": 1, "y": 1, "w": w, "h": h}, {"frame": 0, "x": 3, "y": 0, "w": w, "h": h}]
    dframes = to_dev([frame])
    with Plan(chain(C, "planar"), 2) as p:
        want = [o.reshape(C, h, w).transpose(1, 2, 0) for o in host(p.run(dframes, items))]
    n = w * h * C
    for T, K in ((64, 1), (64, 8), (256, 2), (1024, 1)):
        buf = torch.full((2 * n + 3,), -7.0, dtype=torch.float64, device="cuda:0")
        base = 1 + buf.data_ptr() // 8 % 2  # an odd double: 8-byte aligned
        outs = [buf[base + b * n:base + (b + 1) * n].view(h, w, C) for b in range(2)]
        with Plan(chain(C, "packed"), 2) as p:
            p.set_config(T, K)
            got = host(p.run(dframes, items, outs=outs))
        for b in range(2):
            np.testing.assert_array_equal(got[b].reshape(h, w, C), want[b], err_msg=f"T={T} K={K} item {b}")
        rest = buf.cpu().numpy()
        assert (rest[:base] == -7.0).all() and (rest[base + 2 * n:] == -7.0).all()
