"""Divisions by a constant on the GPU, where their dividends leave the fast
form (subnormals, quotients near the subnormal range) and where zeros,
infinities and NaN pass through it: strict plans give the oracle's bits."""
import numpy as np
import pytest

import fkhelpers as H
import oracle

pytestmark = pytest.mark.gpu

TINY = {"f32": 2.0 ** -149, "f64": 5e-324}
DIVISORS = [1.0, -3.0, 0.229, 255.0, 2.0 ** -149, 2.0 ** -126, 3 * 2.0 ** 100, 3.4e38, float("inf"), 0.0, -0.0]


def frame(dt, h, w, c, g):
    np_dt = np.dtype("f4" if dt == "f32" else "f8")
    v = g.uniform(-300, 300, size=(h, w, c)).astype(np_dt)
    edge = np.array([0.0, -0.0, np.inf, -np.inf, np.nan, TINY[dt], -3 * TINY[dt], np.finfo(np_dt).tiny,
                     np.finfo(np_dt).tiny * 1.5, np.finfo(np_dt).max, 2.0 ** -120], np_dt)
    # the first rows hold ordinary values only (the fast form's waves)
    n = v[h // 2:].size
    pick = g.uniform(size=n) < 0.2
    v[h // 2:].reshape(-1)[pick] = edge[g.integers(0, edge.size, int(pick.sum()))]
    return v


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("c,layout", [(1, "packed"), (3, "planar"), (4, "packed")])
@pytest.mark.parametrize("k", [1, 8])
def test_division_by_constants(dt, c, layout, k):
    g = np.random.default_rng(c * 10 + k)
    fr = frame(dt, 64, 101, c, g)
    item = {"frame": 0, "x": 0, "y": 0, "w": 101, "h": 64}
    for d in DIVISORS:
        per = [float(np.float32(d if i != 1 else 1.5)) for i in range(c)]
        ops = [{"kind": "div", "k": per}, {"kind": "loop", "span": 1, "count": 2}, {"kind": "mul", "k": [0.75]},
               {"kind": "div", "k": [float(np.float32(0.7))]}]
        ch = {"read": {"kind": "plain", "dtype": dt, "channels": c, "out_w": 0, "out_h": 0}, "ops": ops,
              "write": {"dtype": dt, "layout": layout}}
        ref = oracle.run_chain(ch, [fr], [item])[0]["out"]
        with H.Plan(ch, 1, strict=True, tier=1) as p:
            p.set_config(256, k)
            H.assert_bitexact(H.host(p.run(H.to_dev([fr]), [item]))[0], ref, f"{dt} x{c} / {d}")
