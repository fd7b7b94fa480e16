"""The frequencies an at-least-t constraint takes at a point (csrc/eval_kernel.h,
node_window): float64 mirror of the window of the count, the number of
points, the frequencies left out and the coefficients, against the count
recursion, for every restart of a wave sharing one choice."""
import numpy as np
import pytest

B = 42.0
COUNTS = [9 + 8 * i for i in range(16)] + [145 + 16 * i for i in range(8)] + [289 + 32 * i for i in range(8)]


def window(l, k):
    """lo, hi, frac over the restarts (columns) of l [k, R]."""
    lo, hi, frac = k, 0, 0.0
    for c in l.T:
        s1, s = np.sum((1 - c) / 2), np.sum((1 - c * c) / 4)
        a, b = 0, k
        if np.max(np.abs(c)) <= 1 and s > -1:
            v = max(s, 0) + 1e-2
            u = (B / 3 + np.sqrt(B * B / 9 + 2 * B * v)) / v
            for _ in range(2):
                u -= ((1 + u) * np.log1p(u) - u - B / v) / np.log1p(u)
                assert (1 + u) * np.log1p(u) - u >= B / v * (1 - 1e-12)   # Newton stays above the root
            d = u * v + 0.25
            a, b = max(0, int(np.floor(s1 - d))), min(k, int(np.ceil(s1 + d)))
        sm = s - 0.3
        lo, hi = min(lo, a), max(hi, b)
        frac = max(frac, np.arcsin(np.sqrt(B / (2 * sm))) / np.pi if 2 * sm > B else 1.0)
    return lo, hi, frac


def evaluate(l, t, K):
    """Value and gradient of at-least-t as the kernel evaluates them, and the number of frequencies."""
    k, R = l.shape
    lo, hi, frac = window(l, k)
    if t < lo or t > hi + 1:
        return np.full(R, -1.0 if t < lo else 1.0), np.zeros((k, R)), 0
    N = next(c for c in COUNTS if c >= min(hi - lo + 2, k + 1))
    nf = min((N - 1) // 2, (int(frac * N) + 3) & ~1)
    lp = np.concatenate([l, np.ones((K - k, R))])
    val = np.full(R, (2 * (t - lo) - N) / N)
    g = np.zeros((k, R))
    for a in range(1, nf + 1):
        h = np.pi * a / N
        C, tau = np.cos(h), np.tan(h)

        def z(e):
            q = (a * e) % (2 * N)
            return complex(np.cos(np.pi * q / N), np.sin(np.pi * q / N))
        psi = 1 - 1j * tau * lp
        # scaled factors C psi: C^(K-1) of the coefficient with the products
        T = np.prod(C * psi, axis=0)
        c1 = -2.0 / (N * C) * (z(K + 1 - 2 * lo) - z(K + 1 - 2 * t))
        val += (1j * c1 / tau * T).real
        g += (c1 * T / psi[:k]).real
    return val, g, nf


def recursion(l, t):
    """Value and gradient through the count's distribution, in extended precision."""
    k, R = l.shape
    p = ((1 - l) / 2).astype(np.longdouble)
    pre = [np.concatenate([np.ones((1, R)), np.zeros((k, R))]).astype(np.longdouble)]
    for i in range(k):
        d = pre[-1]
        pre.append(d * (1 - p[i]) + np.concatenate([np.zeros((1, R)), d[:-1]]) * p[i])
    back = np.where(np.arange(k + 1)[:, None] >= t, -1.0, 1.0).astype(np.longdouble) * np.ones((1, R))
    g = np.zeros((k, R))
    for i in range(k - 1, -1, -1):
        up = np.concatenate([back[1:], back[-1:]])
        g[i] = np.sum(pre[i] * (back - up), axis=0) / 2
        back = back * (1 - p[i]) + up * p[i]
    return back[0].astype(float), g


def points(k, R, dist, rng):
    u = rng.uniform(-1, 1, (k, R))
    if dist == "settled":
        return np.where(rng.random((k, R)) < 0.8, np.sign(u), u)
    if dist == "corner":
        return np.sign(u)
    if dist == "one_sided":
        return np.clip(np.abs(u) * 0.2 + 0.8, -1, 1)
    if dist == "spread":     # restarts whose counts lie far apart
        return np.clip(u * 0.1 + np.linspace(-0.95, 0.95, R), -1, 1)
    if dist == "outside":
        return u * 1.3
    if dist == "zero":
        return np.zeros((k, R))
    return u


@pytest.mark.parametrize("k,K", [(80, 96), (97, 100), (128, 128), (131, 136), (257, 272), (384, 384), (511, 512), (512, 512)])
@pytest.mark.parametrize("dist", ["uniform", "settled", "corner", "one_sided", "spread", "outside", "zero"])
def test_points_chosen_match_the_recursion(k, K, dist):
    rng = np.random.default_rng(k)
    l = points(k, 4, dist, rng)
    lo, hi, _ = window(l, k)
    # k roundings of terms of modulus at most 1; outside the box the terms grow with prod |l|
    tol = 1e-13 * (1.0 if dist != "outside" else np.prod(np.maximum(1, np.abs(l)), axis=0).max())
    for t in sorted({1, k, max(1, lo - 1), max(1, lo), min(k, lo + 1), (lo + hi + 1) // 2 or 1, min(k, hi), min(k, hi + 1),
                     min(k, hi + 2), k // 4, k // 2}):
        v, g, _ = evaluate(l, t, K)
        rv, rg = recursion(l, t)
        assert np.max(np.abs(v - rv)) <= tol, (t, lo, hi)
        assert np.max(np.abs(g - rg)) <= tol, (t, lo, hi)


def test_points_of_the_box_need_few_frequencies():
    rng = np.random.default_rng(1)
    for dist in ("uniform", "settled", "corner", "one_sided", "zero"):
        for scale in (1.0, 0.7, 0.3):
            l = points(512, 1, dist, rng) * scale
            assert evaluate(l, int(round(np.sum((1 - l) / 2))) or 1, 512)[2] <= 60


def test_point_counts_cover_every_length():
    assert COUNTS[-1] == 513 and all(c % 2 == 1 for c in COUNTS) and COUNTS == sorted(COUNTS)
    # the closed forms of internal.h
    freqs = 0
    for i, c in enumerate(COUNTS):
        cf = 2 * i * (i + 1) if i <= 16 else (544 + (i - 16) * (4 * (i - 16) + 68) if i <= 24 else
                                              1344 + (i - 24) * (8 * (i - 24) + 136))
        assert cf == freqs
        freqs += (c - 1) // 2
    for w in range(1, 514):
        i = 0 if w <= 9 else ((w - 2) >> 3 if w <= 129 else (16 + ((w - 130) >> 4) if w <= 257 else 24 + ((w - 258) >> 5)))
        assert COUNTS[i] >= w and (i == 0 or COUNTS[i - 1] < w)
