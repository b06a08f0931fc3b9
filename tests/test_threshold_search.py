"""CPU emulation of the plain matcher's threshold and list (no device).

A query's candidates come in chunks of 64; the keys (Hamming << 16 | index)
within the threshold are appended to a list of 256 places, which is brought down
to its k smallest when more than 192 are there; too few raise the threshold and
start over.  The threshold is carried to the next query.  Emulated step by step
as the kernel takes them: whatever came before, the threshold stays within the
limit, the list never holds more than its places, the runs are read at most three
times and the k smallest keys inside the limit are found."""
import numpy as np
import pytest

LIST, PASS = 256, 192


def kth_bound(r, K, kk, hG):
    """(bound with exactly kk keys of r within it, its Hamming distance); r: more
    than kk distinct keys, all <= K."""
    r = np.asarray(r)
    count = lambda x: int((r <= x).sum())  # noqa: E731
    upto = lambda h: (h << 16) | 0xFFFF  # noqa: E731
    lo, hi, step, chi = -1, K >> 16, 2, len(r)
    g = min(hG, hi - 1)
    if g >= 0:
        c = count(upto(g))
        if c >= kk:
            hi, chi = g, c
            while hi - step > lo:
                c = count(upto(hi - step))
                if c < kk:
                    lo = hi - step
                    break
                hi, chi = hi - step, c
                step += step
        else:
            lo = g
            while lo + step < hi:
                c = count(upto(lo + step))
                if c >= kk:
                    hi, chi = lo + step, c
                    break
                lo += step
                step += step
    while hi - lo > 1:
        mid = (lo + hi) >> 1
        c = count(upto(mid))
        if c >= kk:
            hi, chi = mid, c
        else:
            lo = mid
    top = min(K, upto(hi))
    if chi == kk:
        return top, hi
    at = hi << 16
    if chi - kk < 8:
        for x in r[(r >= at) & (r <= top)]:
            if count(x) == kk:
                return int(x), hi
    else:
        a, b = at, top
        while a < b:
            mid = a + ((b - a) >> 1)
            c = count(mid)
            if c == kk:
                return mid, hi
            if c < kk:
                a = mid + 1
            else:
                b = mid
    raise AssertionError("no bound found")


class Wave:
    """What a wavefront carries from query to query."""

    def __init__(self, tau, k):
        self.tauK, self.k = (tau << 16) | 0xFFFF, k
        self.hK, self.hG = min(self.tauK, (56 << 16) | 0xFFFF), 52
        self.scans = 0

    def lower(self):
        self.hK = min(self.tauK, max(self.hK, (5 << 16) | 0xFFFF) - 0x10000)

    def query(self, keys, ok):
        total, k = len(keys), self.k
        K = self.hK if total > 64 else self.tauK
        listed, scans = [], 1

        def scan(u0, chunks):
            for i in range(64 * u0, min(64 * (u0 + chunks), total)):
                if ok[i] and keys[i] <= K:
                    listed.append(int(keys[i]))
            assert len(listed) <= LIST

        scan(0, 4)
        if total > 256 or len(listed) > PASS or (len(listed) < k and K != self.tauK):
            u0, again, nch = 4, False, (total + 63) >> 6
            while True:
                while True:
                    if len(listed) > PASS:
                        assert k < len(listed)
                        K, self.hG = kth_bound(listed, K, k, self.hG)
                        listed = [x for x in listed if x <= K]
                        assert len(listed) == k
                        self.lower()
                    if u0 >= nch:
                        break
                    two = 2 if nch - u0 >= 2 and len(listed) <= LIST - 128 else 1
                    scan(u0, two)
                    u0 += two
                if len(listed) >= k or K == self.tauK:
                    break
                K = self.tauK if again else min(self.tauK, K + (6 << 16))
                if not again:
                    self.hK = K
                again = True
                listed.clear()
                u0 = 0
                scans += 1
        assert K <= self.tauK and self.hK <= self.tauK and scans <= 3
        self.scans += scans
        kk = min(len(listed), k)
        if kk and len(listed) > kk:
            bound, self.hG = kth_bound(listed, K, kk, self.hG)
            kept = [x for x in listed if x <= bound]
        else:
            kept = listed
        if len(listed) > 64 and len(listed) > 2 * k:
            self.lower()
        return sorted(kept)


def _query(rng, kind, total):
    """Keys of a query's candidates in the order they are read, and which count
    (a repeat of an earlier table does not)."""
    if kind == "equal":
        h = np.full(total, rng.integers(0, 60))
    elif kind == "falling":
        h = np.linspace(rng.integers(40, 100), 0, total).astype(int)
    elif kind == "crowded":
        h = rng.choice([1, 2, 40, 41], total)
    elif kind == "near":
        h = rng.integers(0, 6, total)
    else:
        h = np.clip(np.rint(64 + 5.7 * rng.standard_normal(total)), 0, 128).astype(int)
    index = rng.permutation(65536)[:total]
    if kind == "equal":
        index = np.sort(index) if rng.random() < 0.5 else np.sort(index)[::-1]
    return (h.astype(np.int64) << 16) | index, rng.random(total) < rng.choice([0.3, 0.9, 1.0])


@pytest.mark.parametrize("tau", [0, 1, 2, 3, 4, 5, 40, 60, 128])
@pytest.mark.parametrize("k", [1, 10, 40, 64])
def test_threshold_search(tau, k):
    rng = np.random.default_rng(1000 * tau + k)
    w = Wave(tau, k)
    for i in range(250):
        kind = rng.choice(["equal", "falling", "crowded", "near", "usual", "usual"])
        total = int(rng.choice([0, 1, 63, 64, 65, 128, 192, 193, 255, 256, 257, 320, 700, 1700]))
        keys, ok = _query(rng, kind, total)
        assert w.hK <= w.tauK
        got = w.query(keys, ok)
        want = np.sort(keys[ok & (keys <= w.tauK)])[:k]
        assert got == want.tolist(), (i, kind, total)

