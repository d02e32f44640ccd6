"""Planar outputs off a 128-byte line, whose stores are ordinary or nontemporal
by the plane's and the launch's bytes and by how the frame is read: a large
launch gives the bits of its items one by one (whose launch is small), and
writes nothing around them."""
import numpy as np
import pytest
import torch

import paper_2508_07071_amd as fk

pytestmark = pytest.mark.gpu


def run(ch, frames, items, out, gap):
    """items' outputs in one tensor, gap values apart, the first one off a line"""
    at = 1
    outs = []
    for it in items:
        shape = fk.out_shape(ch, it)
        k = int(np.prod(shape))
        outs.append(out[at:at + k].view(shape))
        at += k + gap
    h = fk.fk_plan_create(fk.chain_desc(ch), len(items), fk.plan_opts())
    fk.fk_run(h, fk.make_items(ch, frames, items, outs), len(items), fk.stream_handle())
    torch.cuda.synchronize()
    fk.fk_plan_destroy(h)
    return outs


# launches below and above 256 MiB, planes below and above 2 MiB
@pytest.mark.parametrize("w,h,n", [(211, 155, 40), (211, 155, 720), (801, 803, 3), (801, 803, 36)])
@pytest.mark.parametrize("channels", [3, 4])
@pytest.mark.parametrize("offset", [0, 1])  # of the frame: reads by windows or byte by byte
def test_large_launch_equals_single_items(w, h, n, channels, offset):
    ch = {"read": {"kind": "crop_resize", "dtype": "u8", "channels": channels, "out_w": w, "out_h": h},
          "ops": [{"kind": "mul", "k": [1 / 255.0]}], "write": {"dtype": "f32", "layout": "planar"}}
    g = torch.Generator().manual_seed(w)
    size = 300 * 400 * channels
    buf = torch.randint(0, 256, (size + 16,), dtype=torch.uint8, generator=g).cuda()
    frames = [buf[offset:offset + size].view(300, 400, channels)]
    items = [{"frame": 0, "x": 7 * b % 150, "y": 3 * b % 100, "w": 120 + b % 120, "h": 200 - b % 90,
              "out_w": w, "out_h": h} for b in range(n)]
    total = 1 + n * (w * h * channels + 3)
    store = torch.full((total,), -7.0, device="cuda")
    outs = run(ch, frames, items, store, 3)
    one = torch.empty(1 + w * h * channels, device="cuda")
    for b in (0, 1, n // 2, n - 1):
        assert torch.equal(outs[b], run(ch, frames, items[b:b + 1], one, 0)[0]), b
    rest = store[1:].view(n, -1)[:, -3:]
    assert store[0] == -7.0 and bool((rest == -7.0).all())
