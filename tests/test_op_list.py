"""The op list as the kernels run it (fk_chain.cpp lower_ops, built here with
g++): segments of multiply-adds, divisions by a constant and loops.  Run
here in IEEE arithmetic it gives the normalised list's bits, whatever the
ops, loops and constants, and its division forms give the bits of x / d over
the dividends that they accept."""
import os
import struct
import subprocess

import numpy as np
import pytest

import datagen
import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_07071_amd", "csrc")
FMA1, FMAC, FMAR, DIV, LOOP, END = 1, 2, 4, 8, 16, 32
KINDS = {"swap": 0, "cvt": 1, "mul": 2, "add": 3, "sub": 4, "div": 5, "loop": 6}

DRIVER = r"""
#include "fk_chain.hpp"
#include <cstdio>
int main() {
    int C, n, strict, f64;
    while (std::scanf("%d %d %d %d", &C, &n, &strict, &f64) == 4) {
        std::vector<fk_op_desc> ops(n);
        for (auto &o : ops)
            std::scanf("%d %d %a %a %a %a %d %d", &o.kind, &o.n_consts, &o.consts[0], &o.consts[1],
                       &o.consts[2], &o.consts[3], &o.loop_span, &o.loop_count);
        fk_chain_desc ch{};
        ch.read.channels = C;
        ch.ops = ops.data(); ch.n_ops = n;
        std::vector<fk::OpRec> rec;
        int32_t swap = 0;
        fk::normalise_chain(&ch, strict != 0, rec, swap);
        std::vector<uint8_t> prog;
        fk::lower_ops(rec, C, f64 != 0, prog);
        std::printf("%d ", swap);
        for (uint8_t b : prog) std::printf("%02x", b);
        std::printf("\n");
    }
}
"""


@pytest.fixture(scope="module")
def lower(tmp_path_factory):
    d = tmp_path_factory.mktemp("oplist")
    src, exe = str(d / "drv.cpp"), str(d / "drv")
    open(src, "w").write(DRIVER)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-fsanitize=undefined",
                           "-fno-sanitize-recover=undefined", "-I", CSRC, "-o", exe, src,
                           os.path.join(CSRC, "fk_chain.cpp")])

    def run(chains):  # [(ops, C, strict, f64)] -> [(swap, program bytes)]
        lines = []
        for ops, C, strict, f64 in chains:
            lines.append(f"{C} {len(ops)} {int(strict)} {int(f64)}")
            for o in ops:
                k = list(o.get("k", [])) + [0.0] * (4 - len(o.get("k", [])))
                lines.append(f"{KINDS[o['kind']]} {len(o.get('k', []))} " + " ".join(float(v).hex() for v in k)
                             + f" {o.get('span', 0)} {o.get('count', 0)}")
        out = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True,
                             check=True).stdout.split("\n")
        return [(int(ln.split()[0]), bytes.fromhex(ln.split()[1])) for ln in out[:len(chains)]]
    return run


def fma(x, m, a, f64):
    """One rounding of x * m + a: exact products in the wider type.  fp64 is
    evaluated where m or a makes the product or the sum trivial."""
    if f64:
        return np.where(a == 0, x * m, x * m + a)
    return (x.astype(np.float64) * m + a).astype(np.float32)


def div_fast(x, prog, off, c, f64):
    """The division record's fast form, and where the kernel may use it."""
    if f64:
        zh, zl, d = (struct.unpack_from("<d", prog, off + 32 * j + 8 * c)[0] for j in range(3))
        thr = struct.unpack_from("<I", prog, off + 96)[0]
        hi = (x.view(np.uint64) >> 32).astype(np.uint32)
        sub = (x != 0) & (np.abs(x) < 2.0 ** -1022)
    else:
        zh, = struct.unpack_from("<d", prog, off + 8 * c)
        d, = struct.unpack_from("<f", prog, off + 32 + 4 * c)
        thr, = struct.unpack_from("<I", prog, off + 48)
        hi, sub, zl = x.view(np.uint32), np.zeros(x.shape, bool), 0.0
    ok = (((hi << np.uint32(1)) - np.uint32(1)) >= np.uint32(thr)) & ~sub
    return zh, zl, d, ok


def run_program(x, C, swap, prog, f64):
    V, es = (np.float64, 8) if f64 else (np.float32, 4)
    x = x.astype(V).reshape(-1, C)
    if swap and C >= 3:
        x = x[:, [2, 1, 0] + list(range(3, C))]
    const = lambda off, n: np.frombuffer(prog, V, n, off)  # noqa: E731
    i, runs = 0, 1
    while True:
        kind, n, off, reps = struct.unpack_from("<iiIi", prog, 16 * i)
        i += 1
        if kind == END:
            return x
        if kind == LOOP:
            if runs < reps:
                runs, i = runs + 1, i - n - 1
            else:
                runs = 1
        elif kind == FMA1:
            for r in range(n):
                m, a = const(off + 2 * es * r, 2)
                x = fma(x, m, a, f64)
        elif kind in (FMAC, FMAR):
            for r in range(n if kind == FMAC else reps):
                k = const(off + (8 * es * r if kind == FMAC else 0), 8)
                x = fma(x, k[:C], k[4:4 + C], f64)
        else:
            for _ in range(reps):
                cols = []
                for c in range(C):
                    zh, zl, d, ok = div_fast(x[:, c].copy(), prog, off, c, f64)
                    q = x[:, c] / V(d)
                    if not f64:  # fp64's form is checked in exact arithmetic below
                        q = np.where(ok, (x[:, c].astype(np.float64) * zh).astype(np.float32), q)
                    cols.append(q)
                x = np.stack(cols, 1)


def random_ops(g, C, n):
    ops, run = [], 0
    for _ in range(n):
        kind = ["swap", "cvt", "mul", "add", "sub", "div"][int(g.integers(0, 6))]
        k = []
        if kind in ("mul", "div", "add", "sub"):
            lo, hi = (0.5, 1.5) if kind in ("mul", "div") else (-1.0, 1.0)
            k = [datagen.f32(g.uniform(lo, hi)) for _ in range(1 if g.uniform() < 0.5 else C)]
        ops.append({"kind": kind, "k": k})
        run = run + 1 if k else 0
        if run and g.uniform() < 0.2:
            ops.append({"kind": "loop", "span": int(g.integers(1, run + 1)), "count": int(g.integers(1, 5))})
            run = 0
        elif run and g.uniform() < 0.15:
            ops += [dict(ops[-1])] * int(g.integers(1, 4))  # identical records
            run += 1
    return ops


@pytest.mark.parametrize("C", [1, 3, 4])
def test_program_gives_the_chain_bits(lower, C):
    """Strict lists of every mix, loop and length (runs of 1..9 multiply-adds
    among them) against the oracle's unfused chain, bit for bit."""
    g = datagen.rng(40 + C)
    cases = [random_ops(g, C, n) for n in list(range(0, 12)) + [17, 31, 64] * 6]
    frames = [(g.uniform(-300, 300, size=(5, 7, C)) * (g.uniform(size=(5, 7, C)) < 0.9)).astype(np.float32)
              for _ in cases]  # a tenth of the values are (signed) zeros
    for ops, fr, (swap, prog) in zip(cases, frames, lower([(o, C, True, False) for o in cases])):
        ch = {"read": {"kind": "plain", "dtype": "f32", "channels": C, "out_w": 0, "out_h": 0}, "ops": ops,
              "write": {"dtype": "f32", "layout": "packed"}}
        ref = oracle.run_chain(ch, [fr], [{"frame": 0, "x": 0, "y": 0, "w": 7, "h": 5}])[0]["out"]
        got = run_program(fr, C, swap, prog, False).reshape(ref.shape)
        np.testing.assert_array_equal(got.view(np.uint32), ref.view(np.uint32))


def test_segments(lower):
    mul, add, div = ({"kind": k, "k": [v]} for k, v in (("mul", 2.0), ("add", 3.0), ("div", 4.0)))
    per = {"kind": "sub", "k": [1.0, 2.0, 3.0]}
    loop = lambda s, c: {"kind": "loop", "span": s, "count": c}  # noqa: E731
    cases = [([mul, add, div, add, per], [FMA1, DIV, FMAC]),
             ([mul, add, loop(2, 5), mul], [FMA1, LOOP, FMA1]),
             ([add, mul, div, loop(2, 3)], [FMA1, FMA1, DIV, LOOP]),
             ([mul, loop(1, 6), add], [FMAR, FMA1]), ([div, div, div], [DIV]), ([], [])]
    for (ops, want), (_, prog) in zip(cases, lower([(o, 3, True, False) for o, _ in cases])):
        kinds, i = [], 0
        while struct.unpack_from("<i", prog, 16 * i)[0] != END:
            kinds.append(struct.unpack_from("<i", prog, 16 * i)[0])
            i += 1
        assert kinds == want, (ops, kinds)


EDGE = np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 2.0 ** -149, -3 * 2.0 ** -149, 2.0 ** -126, 1.5 * 2.0 ** -126,
                 2.0 ** -125, 3 * 2.0 ** -120, 2.0 ** 127, 3.4e38, 1.0, -255.0], np.float32)
DIVISORS = [1.0, -1.0, 3.0, 0.229, 1.5, 255.0, 2.0 ** -149, 5 * 2.0 ** -140, 2.0 ** -126, 3 * 2.0 ** 120, 3.4e38,
            float("inf"), float("-inf"), 0.0, -0.0, 1.9999999, 0.50000006]


def test_fp32_division_form_is_exact(lower):
    """(float)((double)x * RN64(1 / d)) against x / d for random and edge
    dividends and divisors of every exponent."""
    g = datagen.rng(3)
    ds = [float(np.float32(d)) for d in DIVISORS] + \
         [float(v) for v in (g.uniform(1, 2, 300).astype(np.float32) * (2.0 ** g.integers(-126, 127, 300))
                             .astype(np.float32) * g.choice([-1, 1], 300)).astype(np.float32)]
    ops = [[{"kind": "div", "k": [d]}] for d in ds]
    x = np.concatenate([EDGE, g.integers(0, 2 ** 32, 20000, dtype=np.uint64).astype(np.uint32).view(np.float32),
                        g.integers(0, 256, 4000).astype(np.float32), g.uniform(-4, 4, 20000).astype(np.float32)])
    with np.errstate(all="ignore"):
        for d, (_, prog) in zip(ds, lower([(o, 1, True, False) for o in ops])):
            off, = struct.unpack_from("<I", prog, 8)
            zh, _, dd, ok = div_fast(x, prog, off, 0, False)
            assert np.float32(dd).tobytes() == np.float32(d).tobytes()
            # quotients next to a rounding boundary: x = the fp32 values around m * d, m a midpoint
            m = (g.integers(2 ** 24, 2 ** 25, 4000) | 1).astype(np.float64) * 2.0 ** -24
            near = np.nextafter((m * d).astype(np.float32), g.choice([-np.inf, np.inf], 4000).astype(np.float32))
            for xs in (x, near, (m * d).astype(np.float32)):
                _, _, _, ok = div_fast(xs, prog, off, 0, False)
                q, ref = (xs.astype(np.float64) * zh).astype(np.float32), xs / np.float32(d)
                same = (q.view(np.uint32) == ref.view(np.uint32)) | (np.isnan(q) & np.isnan(ref))
                assert np.all(same | ~ok), (d, xs[~same & ok][:3])
            # zeros and ordinary dividends by ordinary divisors take the form
            ok = div_fast(x, prog, off, 0, False)[3]
            assert ok[x == 0].all() and (not 0.5 < abs(d) < 2.0 ** 24 or ok[np.abs(x) >= 1.0].all())


def test_fp64_division_form_is_exact(lower):
    """fma(x, zh, x * zl) in exact rational arithmetic against x / d; zeros,
    infinities and NaN are v_div_fixup's."""
    from fractions import Fraction
    g = datagen.rng(4)
    ds = [d for d in (float(np.float32(d)) for d in DIVISORS) if np.isfinite(d) and d != 0.0] + \
         [float(np.float32(v)) for v in g.uniform(0.5, 1.5, 60)]
    edge = [5e-324, -5e-324, 1e-310, 2.0 ** -1040, 2.0 ** -1022, 2.0 ** -1000, 2.0 ** -900, 1e-200, 1.0, 255.0,
            1e300, 1.7e308, -3.5]
    for d, (_, prog) in zip(ds, lower([([{"kind": "div", "k": [d]}], 1, True, True) for d in ds])):
        off, = struct.unpack_from("<I", prog, 8)
        m = (int(g.integers(2 ** 53, 2 ** 54)) | 1) * 2.0 ** -53
        xs = np.array(edge + list(g.uniform(-300, 300, 60)) + [m * d, np.nextafter(m * d, 9e9)], np.float64)
        zh, zl, dd, ok = div_fast(xs, prog, off, 0, True)
        assert dd == d
        for x, good in zip(xs, ok):
            if not good:
                continue
            # x * zl rounded, then the exact fma rounded once
            try:
                q = float(Fraction(float(x)) * Fraction(zh) + Fraction(float(x) * zl))
            except OverflowError:
                q = np.copysign(np.inf, x * d)
            with np.errstate(over="ignore"):
                assert q == np.float64(x) / np.float64(d), (x, d)
        assert not ok[:4].any()  # subnormals take the general division
