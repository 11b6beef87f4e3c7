"""The rounds of the boundary search over compressed levels (group_search) on the CPU, with its sample placement in single
precision: samples ascend and lie in their windows up to windows of 2^31 - 1 entries, and the search ends at the boundary of
Algorithm 1 after few rounds, for operands spread nothing alike."""
import bisect
import random

import numpy as np
import pytest

f32 = np.float32
LANES = {1: 64, 2: 32, 3: 21, 4: 16, 5: 12, 6: 10, 7: 9, 8: 8}
SPACE = 2**31 - 1


def _sample(i, size, w, at, even):
    """aimed_sample: the place of sample i of `size` in a window of w entries, the boundary expected `at` entries in."""
    inv, whole = f32(2) * (f32(1) / f32(size - 1)), f32(w)
    e = f32(i) * inv - f32(1)
    x = f32(0.5) * (whole + whole * e)
    if not even:
        left, right = max(f32(at), f32(1)), max(whole - f32(at), f32(1))
        near = max(f32(0.5) * np.sqrt(left * right * (f32(1) / (left + right))), f32(0.5))
        side = max(left if e < 0 else right, near)
        off = near * np.exp2(abs(e) * np.log2(side * (f32(1) / near)))
        x = f32(at) if abs(e) * f32(size) < f32(0.5) else f32(at) + np.copysign(off, e)
    s = min(int(min(max(x, f32(0)), min(whole, f32(2147483520)))), w - 1)
    return 0 if i == 0 else w - 1 if i == size - 1 else s


class _Rows:
    """n ascending coordinates, the i-th by a function."""

    def __init__(self, n, f):
        self.n, self.at = n, f

    def before(self, x):
        lo, hi = 0, self.n
        while lo < hi:
            mid = (lo + hi) // 2
            lo, hi = (mid + 1, hi) if self.at(mid) < x else (lo, mid)
        return lo


def _search(ops, R):
    """(coordinate, positions, rounds, rounds that looked up a middle entry)"""
    k, size = len(ops), LANES[len(ops)]
    lo, hi = [0] * k, [o.n for o in ops]
    W, even, middles = sum(hi), False, 0
    share = f32(R) / f32(W)
    for rounds in range(1, 1100):
        wide = [hi[t] - lo[t] > size for t in range(k)]

        def place(t, even):
            w = hi[t] - lo[t]
            return [_sample(i, size, w, f32(0) if even is None else share * f32(w), even is None or even)
                    for i in range(size)] if wide[t] else list(range(w))

        S = [place(t, even) for t in range(k)]
        if any(a > b for s in S for a, b in zip(s, s[1:])):
            S = [place(t, None) for t in range(k)]
        for t in range(k):
            assert all(a <= b for a, b in zip(S[t], S[t][1:])) and all(0 <= a < hi[t] - lo[t] for a in S[t])
        V = [[ops[t].at(lo[t] + a) for a in S[t]] for t in range(k)]
        left, below, above = R - sum(lo), -1, None
        for t in range(k):
            for a, v in zip(S[t], V[t]):
                least = most = a
                for u in range(k):
                    if u != t:
                        c = bisect.bisect_left(V[u], v)
                        behind = S[u][c - 1] + 1 if c else None
                        ahead = S[u][c] if c < len(S[u]) else hi[u] - lo[u]
                        least += behind if c else ahead
                        most += behind if c == size else ahead
                if most <= left:
                    below = max(below, v)
                if least > left:
                    above = v if above is None else min(above, v)
        new_lo, new_hi = [], []
        for t in range(k):
            c1 = bisect.bisect_left(V[t], below)
            c2 = len(V[t]) if above is None else bisect.bisect_left(V[t], above)
            hit = c1 < len(V[t]) and V[t][c1] == below
            new_lo.append(lo[t] + (S[t][c1] if hit else S[t][c1 - 1] + 1 if c1 else 0))
            new_hi.append(hi[t] if c2 == len(V[t]) else lo[t] + S[t][c2])
        if not any(wide):
            return below, new_lo, rounds, middles
        lo, hi = new_lo, [max(a, b) for a, b in zip(new_hi, new_lo)]
        now = sum(hi) - sum(lo)
        slow = now > W - (W >> 2) if even else now > W >> 1
        if slow and even:
            middles += 1
            t = max(range(k), key=lambda u: hi[u] - lo[u])
            mid = ops[t].at(lo[t] + ((hi[t] - lo[t]) >> 1))
            at = [ops[u].before(mid) for u in range(k)]
            if sum(at) <= R:
                lo = at
            else:
                hi = at
            now = sum(hi) - sum(lo)
        even, W = slow and not even, now
        share = f32(R - sum(lo)) / f32(now) if now else f32(0)
    raise AssertionError("no end")


def _operand(rng, kind, k):
    n = rng.choice([5, 70, 1000, 10**5, 10**7])
    if kind == "full":                                  # together as many entries as there may be
        return _Rows(SPACE // k - rng.randrange(1000), lambda i: i)
    if kind == "power":
        p = rng.uniform(0.05, 8)
        return _Rows(n, lambda i: int((SPACE - n) * ((i / n) ** p)) + i)
    if kind == "halves":                                # both ends of the space
        q = rng.random()
        return _Rows(n, lambda i: i if i < q * n else SPACE - n + i)
    if kind == "inside":                                # the first and the last coordinate, the rest in the middle
        return _Rows(n, lambda i: 0 if i == 0 else SPACE - 1 if i == n - 1 else SPACE // 2 + i)
    n = rng.choice([LANES[k] + 1, LANES[k] + 2, 2 * LANES[k], 300])       # "short": windows a little longer than the lanes
    at = sorted(rng.sample(range(rng.choice([2 * n, 40 * n, 10**6])), n))
    return _Rows(n, lambda i: at[i])


@pytest.mark.parametrize("kind", ["full", "power", "halves", "inside", "short"])
@pytest.mark.parametrize("k", range(1, 9))
def test_rounds(k, kind):
    rng = random.Random(f"{k} {kind}")
    for _ in range(12):
        ops = [_operand(rng, kind, k) for _ in range(k)]
        total = sum(o.n for o in ops)
        for R in (0, total - 1, rng.randrange(total), rng.randrange(total)):
            x, at, rounds, middles = _search(ops, R)
            assert at == [o.before(x) for o in ops] and sum(at) <= R < sum(o.before(x + 1) for o in ops)
            # (evenly spaced samples leave four of the size - 1 gaps, 4/7 at most: no look-up of a middle entry)
            assert rounds <= 24 and middles == 0, (rounds, middles)


@pytest.mark.parametrize("size", sorted(LANES.values()))
def test_samples_of_large_windows(size):
    """Where floats are further apart than the entries: what does not ascend is caught, evenly spaced samples always do."""
    rng = random.Random(size)
    for _ in range(300):
        w = rng.choice([size + 1, 2**24 + 1, 2**31 - 1, rng.randrange(size + 1, 2**31)])
        at = f32(rng.random()) * f32(w)
        aimed = [_sample(i, size, w, at, False) for i in range(size)]
        spread = [_sample(i, size, w, 0, True) for i in range(size)]
        assert all(0 <= a < w for a in aimed + spread) and spread == sorted(spread)
        assert spread[0] == aimed[0] == 0 and spread[-1] == aimed[-1] == w - 1
