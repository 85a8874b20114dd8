"""The clash arcs' ends (host arithmetic, no GPU): the search kernel's polynomials, read from its source,
stay within its stated 8e-5 turns of the exact angle for |t| <= 0.9995, with the hardware's square root,
reciprocal and reciprocal square root off by an ulp either way; the guard around whole turns (2e-4), inside
which the kernel takes the library functions, is wider than that and both functions' errors together."""
import os
import re

import numpy as np

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2110_11644_amd", "csrc",
                   "dock_kernels.inc")
f32, TWO_PI = np.float32, 2 * np.pi


def source():
    text = open(SRC).read()
    at = text.index("void clash_arc(")
    return text[at:text.index("flush_arcs", at)]


def horner(body, var, x):
    """The polynomial p (or h) of the kernel in its own FP32 steps (a fused multiply-add rounds once)."""
    coef = r"(-?\d\.\d+)f"
    first = re.search(r"float %s = fmaf\(\w, %s, %s\);" % (var, coef, coef), body)
    rest = re.findall(r"^\s*%s = fmaf\(\w, %s, %s\)" % (var, var, coef), body, re.M)
    assert first and len(rest) == 4
    x = f32(x)
    acc = f32(np.float64(x) * np.float64(f32(first.group(1))) + np.float64(f32(first.group(2))))
    for c in rest:
        acc = f32(np.float64(x) * np.float64(acc) + np.float64(f32(c)))
    return acc


def ulp(v, by):
    return v if by == 0 else np.nextafter(v, f32(np.inf if by > 0 else -np.inf))


def ends(body, dA, B, C, by, S):
    """lo, hi of the kernel in turns, and t; by: errors in ulp of rsq, sqrt and rcp."""
    k = f32(S / 6.283185307179586)
    pi = f32(3.14159265)
    R2 = f32(np.float64(B) * B + np.float64(f32(np.float64(C) * C)))
    t = f32(-dA * ulp(f32(1 / np.sqrt(np.float64(R2))), by[0]))
    x = np.abs(t)
    p = f32(horner(body, "p", x) * ulp(f32(np.sqrt(np.maximum(np.float64(f32(f32(1) - x)), 0))), by[1]))
    alpha = np.where(t < 0, f32(pi - p), p)
    ab, ac = np.abs(B), np.abs(C)
    q = f32(np.minimum(ab, ac) * ulp(f32(1 / np.float64(np.maximum(ab, ac))), by[2]))
    h = f32(horner(body, "h", f32(q * q)) * q)
    h = np.where(ac > ab, f32(f32(0.5) * pi - h), h)
    h = np.where(B < 0, f32(pi - h), h)
    phi = np.copysign(h, C)
    lo = f32(f32(phi + alpha) * k)
    hi = f32(f32(f32(phi + f32(f32(2) * pi)) - alpha) * k)
    return lo, hi, t


def test_ends_within_their_bound():
    body = source()
    limit = float(re.search(r"x <= (0\.\d+)f", body).group(1))
    guard = 0.5 - float(re.search(r"- 0\.5f\) < (0\.\d+)f", body).group(1))
    assert limit == 0.9995 and abs(guard - 2e-4) < 1e-9
    rng = np.random.default_rng(17)
    n = 400000
    t = np.concatenate([rng.uniform(-0.9995, 0.9995, n), np.linspace(-0.9995, 0.9995, 20001),
                        np.sign(rng.uniform(-1, 1, n)) * (0.9995 - 10.0 ** rng.uniform(-7, -1, n))])
    phi = rng.uniform(-np.pi, np.pi, t.size)
    phi[::7] = np.round(phi[::7] * 4 / np.pi) * np.pi / 4 + rng.normal(0, 1e-4, phi[::7].size)
    R = 10.0 ** rng.uniform(-2, 3, t.size)
    B, C, dA = f32(R * np.cos(phi)), f32(R * np.sin(phi)), f32(-R * t)
    te = -dA.astype(np.float64) / np.hypot(B.astype(np.float64), C)
    S, worst = 32, 0.0
    for by in [(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1)]:
        lo, hi, tk = ends(body, dA, B, C, by, S)
        use = np.abs(tk) <= f32(limit)
        alpha, ph = np.arccos(np.clip(te, -1, 1)), np.arctan2(C.astype(np.float64), B)
        for got, want in ((lo, ph + alpha), (hi, ph + TWO_PI - alpha)):
            worst = max(worst, np.abs(got - want * S / TWO_PI)[use].max())
    print("worst %.3g turns of 1 / 32" % worst)
    assert worst <= 8e-5
    # the library functions' own ends: a few ulp of angles below 3 pi, and t's two roundings near 1
    library = (6 * 2.0 ** -24 * 9.43 + 3 * 2.0 ** -24 / np.sqrt(1 - limit ** 2)) * S / TWO_PI
    assert worst + library < guard
