"""The dense walk and its count pass.  Boundary times: the reciprocal form n y with two FMA corrections gives the rounded
quotient n / w (emulated here in exact rationals, an FMA rounding once), over the operands that the
walk admits: w of magnitude in [2^-100, 2^100) with a significand below 2 - 2^-48, n zero or of
magnitude in [2^-900, 2^900)."""
import math
import random
from fractions import Fraction as Q

import pytest


def fma(a, b, c):
    return float(Q(a) * Q(b) + Q(c))


def quot(n, w):
    y = 1.0 / w
    q0 = n * y
    q1 = fma(fma(-w, q0, n), y, q0)
    return fma(fma(-w, q1, n), y, q1)


def _sig(rng, kind):
    """A significand in [1, 2): random, next to 1, next to 2 - 2^-48, or of few bits."""
    top = 2 ** 52 - 17
    if kind == 0:
        k = rng.randrange(top + 1)
    elif kind == 1:
        k = rng.randrange(64)
    elif kind == 2:
        k = top - rng.randrange(64)
    else:
        k = sum(1 << rng.randrange(52) for _ in range(2)) % (top + 1)
    return 1.0 + k * 2.0 ** -52


@pytest.mark.parametrize("exps", [(-3, 3), (-100, 99)])
def test_reciprocal_quotient_is_the_division(exps):
    rng = random.Random(5)
    for t in range(12000):
        w = _sig(rng, t % 4) * 2.0 ** rng.randint(*exps) * rng.choice((1, -1))
        if t % 5 == 0:     # numerators next to a product of w: quotients next to a tie or exact
            n = w * _sig(rng, (t // 4) % 4)
            n = n * (1 + rng.randint(-3, 3) * 2.0 ** -52)
        else:
            n = _sig(rng, (t // 4) % 4) * 2.0 ** rng.randint(-900 if exps[0] < -50 else -9, 899 if exps[0] < -50 else 9)
        n *= rng.choice((1, -1))
        assert quot(n, w) == n / w, (n.hex(), w.hex())
    assert quot(0.0, 1.7) == 0.0 and quot(0.0, -1.7) == 0.0


# ---- the number of voxels from the faces crossed along each axis

def _ray(rng, kind, n, h, o):
    """A ray (centre, direction, start, end) of the grid; kinds that share boundary times come from
    centres on the lattice and directions of few bits, equal or integer multiples of each other."""
    c = [o[a] + rng.uniform(-0.3, 1.3) * n[a] * h for a in range(3)]
    w = [rng.uniform(-1, 1) for _ in range(3)]
    if kind == 1:     # lattice centre, simple slopes
        c = [o[a] + h * rng.randrange(-2, n[a] + 3) for a in range(3)]
        w = [rng.choice((1.0, 0.5, 0.25, 0.75)) * rng.choice((1, -1)) for _ in range(3)]
    elif kind == 2:   # two equal slopes, a parallel axis now and then
        w[1] = rng.choice((1, -1)) * w[0]
        c[1] = o[1] + rng.choice((1, -1)) * (c[0] - o[0])
        if rng.random() < 0.3:
            w[2] = 0.0
    elif kind == 3:   # almost parallel to an axis
        w[rng.randrange(3)] *= 2.0 ** -rng.randrange(5, 40)
    elif kind == 4:   # almost shared times
        w[1] = w[0] * (1 + rng.randint(-4, 4) * 2.0 ** -rng.choice((22, 30, 50, 52)))
        c[1] = o[1] + (c[0] - o[0]) * (1 + rng.randint(-4, 4) * 2.0 ** -rng.choice((22, 30, 50, 52)))
    ts, te = 0.0, float("inf")
    for a in range(3):
        lo, hi = o[a], o[a] + n[a] * h
        if w[a] == 0.0:
            if not lo <= c[a] < hi:
                return None
            continue
        t0, t1 = (lo - c[a]) / w[a], (hi - c[a]) / w[a]
        ts, te = max(ts, min(t0, t1)), min(te, max(t0, t1))
    if rng.random() < 0.7:
        te = min(te, ts + rng.random() * (te - ts))
    return (c, w, ts, te) if te > ts else None


def _first(n, h, o, c, w, ts, a):
    q = math.floor((c[a] + ts * w[a] - o[a]) / h)
    return float(min(max(q, 0), n[a] - 1))


def _start(n, h, o, ray):
    """State before the first chord: face numbers and times of the axes, entry time, chords so far."""
    c, w, ts, te = ray
    f, t = [0.0] * 3, [float("inf")] * 3
    for a in range(3):
        f[a] = _first(n, h, o, c, w, ts, a) + (w[a] > 0)
        if w[a] != 0.0:
            t[a] = ((o[a] + f[a] * h) - c[a]) / w[a]
    return f, t, ts, 0


def _chords(n, h, o, ray, state, tend=float("inf")):
    """(number, last face of each axis, t_in, t_out) of the chords from a state on that end by tend."""
    c, w, ts, te = ray
    f, t, tin, k = list(state[0]), list(state[1]), state[2], state[3]
    out = []
    while True:
        a = min(range(3), key=lambda i: t[i])   # the lowest axis of a tie
        if t[a] > tend:
            return out
        if min(t[a], te) > tin:
            out.append((k, tuple(f), tin, min(t[a], te)))
            k += 1
        if t[a] >= te:
            return out
        tin = max(tin, t[a])
        f[a] += 1.0 if w[a] > 0 else -1.0
        t[a] = ((o[a] + f[a] * h) - c[a]) / w[a]


def _walk(n, h, o, ray):
    return len(_chords(n, h, o, ray, _start(n, h, o, ray)))


def _parts(n, h, o, ray, parts=4):
    """The chords by quarters of the ray, each from the faces before it (None: not split)."""
    c, w, ts, te = ray

    def cut(p):
        return ts + (te - ts) * (p * (1.0 / parts))
    if not (cut(1) > ts and cut(parts - 1) < te) or _faces(n, h, o, ray) < 0:
        return None
    out = []
    for p in range(parts):
        f, t, tin, k = _start(n, h, o, ray)
        for a in range(3):
            if p == 0 or w[a] == 0.0:
                continue
            s, f0, tau = (1.0 if w[a] > 0 else -1.0), f[a], cut(p)

            def time(x):
                return ((o[a] + x * h) - c[a]) / w[a]
            m = int(min(max(math.floor((((c[a] + tau * w[a]) - o[a]) / h - f0) * s) + 1.0, 0.0), 1024.0))
            if m > 0 and time(f0 + s * (m - 1)) > tau:
                m -= 1
            elif time(f0 + s * m) <= tau:
                m += 1
            if m == 0:
                continue
            k += m - 1 if t[a] <= ts else m
            tin = max(tin, time(f0 + s * (m - 1)))
            f[a] = f0 + s * m
            t[a] = time(f[a])
        out += _chords(n, h, o, ray, (f, t, tin, k), cut(p + 1) if p < parts - 1 else float("inf"))
    return out


def _faces(n, h, o, ray):
    c, w, ts, te = ray
    rh = 1.0 / h
    cnt, t0, y = [0] * 3, [0.0] * 3, [0.0] * 3
    mh = [(abs(o[a]) + abs(c[a])) * rh + (n[a] + 2) for a in range(3)]
    if not max(mh) < 2.0 ** 25:
        return -1
    for a in range(3):
        if w[a] == 0.0:
            continue
        s = 1.0 if w[a] > 0 else -1.0
        f0 = _first(n, h, o, c, w, ts, a) + (w[a] > 0)
        y[a] = 1.0 / w[a]

        def time(f):
            return ((o[a] + f * h) - c[a]) / w[a]
        e = math.ceil((((c[a] + te * w[a]) - o[a]) * rh - f0) * s)
        if e > 1024:
            return -1
        m = max(e, 0)
        if m > 0 and time(f0 + s * (m - 1)) >= te:
            m -= 1
        elif time(f0 + s * m) < te:
            m += 1
        if m == 0:
            continue
        t0[a] = time(f0)
        if t0[a] <= ts:
            m -= 1
            t0[a] = time(f0 + s)
            if t0[a] <= ts:
                return -1
        cnt[a] = m
    for p, q in ((0, 1), (0, 2), (1, 2)):
        if cnt[q] < cnt[p]:
            p, q = q, p
        if cnt[p] == 0:
            continue
        a = w[q] * abs(y[p])
        if not mh[p] * abs(a) + mh[q] < 2.0 ** 25:
            return -1
        g = ((c[q] + t0[p] * w[q]) - o[q]) * rh
        x = int((g - math.floor(g)) * 2.0 ** 32) + 2048
        dx = int((a - math.floor(a)) * 2.0 ** 32)
        if min((x + k * dx) & 0xffffffff for k in range((cnt[p] + 7) // 8 * 8)) <= 4096:
            return -1
    return sum(cnt) + 1


@pytest.mark.parametrize("n,h,o", [((25, 25, 15), 0.2, (-2.5, -2.5, -0.3)), ((250, 240, 150), 0.02, (-2.5, 1.1, 0.0)),
                                   ((1, 7, 64), 0.25, (0.0, -0.875, 8.0)), ((2000, 3, 3), 0.01, (100.0, -0.01, 0.0))])
def test_voxels_counted_by_faces_are_those_walked(n, h, o):
    rng = random.Random(11)
    for kind in range(5):
        rays = [r for r in (_ray(rng, kind, n, h, o) for _ in range(1200)) if r]
        got = [_faces(n, h, o, r) for r in rays]
        for r, g in zip(rays, got):
            assert g < 0 or g == _walk(n, h, o, r), (kind, r)
        if kind == 0:   # rays at random are counted: a shared time is seen in one of 8192
            assert max(n) > 1024 or sum(g < 0 for g in got) <= 0.01 * len(got)
        if kind == 1 and min(n) > 1:   # shared times are found
            assert sum(g < 0 for g in got) > 0.2 * len(got)


@pytest.mark.parametrize("n,h,o", [((25, 25, 15), 0.2, (-2.5, -2.5, -0.3)), ((250, 240, 150), 0.02, (-2.5, 1.1, 0.0)),
                                   ((1, 7, 64), 0.25, (0.0, -0.875, 8.0))])
def test_chords_by_parts_are_those_walked(n, h, o):
    rng = random.Random(12)
    for kind in range(5):
        rays = [r for r in (_ray(rng, kind, n, h, o) for _ in range(500)) if r]
        split = 0
        for r in rays:
            if rng.random() < 0.2:   # an end next to the start
                r = (*r[:3], r[2] + (r[3] - r[2]) * 2.0 ** -rng.randrange(1, 52))
                if r[3] <= r[2]:
                    continue
            got = _parts(n, h, o, r)
            if got is not None:
                split += 1
                assert got == _chords(n, h, o, r, _start(n, h, o, r)), (kind, r)
        assert split > 0.9 * len(rays) * 0.8 if kind == 0 else True
