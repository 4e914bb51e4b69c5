"""The records behind the list build's matrix-core pair tests, on the CPU.

Offsets form (n_cell >= 3): the 16 f16 slots of a candidate (its own offset,
no shift) and of a home atom shifted by the row's offset are exact in f16 and
their products accumulated in f32 in any order give 1/2 - S exactly, at the
extremes the kernel admits.  Circle form (n_cell <= 2): with slots rounded to
f16 the entry stays negative for every pair within its list radius, at the
radius itself, for boxes down to the smallest the library takes."""
import numpy as np
import pytest


def cand_slots(q, C, d):
    s = np.zeros(16)
    s[:4] = [2 * q[d - 1], 2048, 1, 1]
    s[4:d + 3] = 2 * q[:d - 1]
    s[d + 3:d + 5] = [C >> 11, C & 2047]
    return s


def home_slots(q, o, T, d):
    qp = q - 250 * o
    B = int(qp @ qp) - T
    s = np.zeros(16)
    s[:4] = [-qp[d - 1], B >> 11, B & 2047, 0.5]
    s[4:d + 3] = -qp[:d - 1]
    s[d + 3:d + 5] = [-2048, -1]
    return s, qp, B


@pytest.mark.parametrize("d", [2, 6, 10])
@pytest.mark.parametrize("reach", [1, 2])
def test_offset_slots_exact(d, reach):
    g = np.random.default_rng(10 * d + reach)
    Tmax = int(2 * (125 * reach + np.sqrt(d) / 2 * 1.000001) ** 2) + 1
    for _ in range(300):
        q, p = g.integers(-127, 128, d), g.integers(-127, 128, d)
        o = g.integers(-reach, reach + 1, d)
        Ti, Tj = (int(g.integers(1, Tmax + 1)) for _ in range(2))
        if g.random() < 0.3:
            q, p = g.choice([-127, 127], d), g.choice([-127, 127], d)
            o, Ti, Tj = g.choice([-reach, reach], d), Tmax, Tmax
        C = Tj - int(p @ p)
        a = cand_slots(p, C, d)
        b, qp, B = home_slots(q, o, Ti, d)
        for v in (a, b):
            assert np.array_equal(v.astype(np.float16).astype(np.float64), v)
        S = int(qp @ (2 * p)) + C - B
        assert (S > 0) == (int(((p - qp) ** 2).sum()) < Ti + Tj)
        prods = (a * b).astype(np.float32)
        assert np.array_equal(prods.astype(np.float64), a * b)
        for _ in range(3):
            acc = np.float32(0.0)
            for t in prods[g.permutation(16)]:
                acc = np.float32(acc + t)
            assert float(acc) == 0.5 - S


@pytest.mark.parametrize("d", range(2, 11))
@pytest.mark.parametrize("frac", [0.34, 0.5, 0.62, 0.9])
def test_circle_slots_keep_every_pair(d, frac):
    """frac: largest list radius over the box side."""
    g = np.random.default_rng(d)
    L = 3.7
    margin = d * (1.42 / 2048.0 + 2.0 / 2048.0)
    m = 4000
    ai, aj = (g.uniform(0.7, 1.0, m) * 0.5 * frac * L for _ in range(2))
    v = g.normal(size=(m, d))
    v[: m // 4] *= g.uniform(size=(m // 4, d)) < 0.3   # along few axes too
    v[np.abs(v).sum(1) == 0, 0] = 1.0
    r = (ai + aj) * np.where(g.uniform(size=m) < 0.5, 1.0 - 1e-12, g.uniform(size=m))
    x = g.uniform(-L / 2, L / 2, (m, d))
    y = x + r[:, None] * v / np.linalg.norm(v, axis=1, keepdims=True)

    def rec(p):
        th = (p / L * 2 * np.pi).astype(np.float32)
        e = np.stack([np.cos(th), np.sin(th)], -1).astype(np.float16)
        return e.reshape(m, -1).astype(np.float32)

    def share(a):
        t = np.maximum(0.5 * d - (2 * np.pi / L * a) ** 2 - margin, -2.0 * d)
        return t.astype(np.float32).astype(np.float16).astype(np.float32)

    entry = share(ai) + share(aj) - (rec(x) * rec(y)).sum(1, dtype=np.float32)
    assert (entry < 0).all()
