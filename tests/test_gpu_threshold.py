"""The matcher's threshold and its list of candidates against the oracle, bit for
bit, on codes and keys made for them: equal keys make every train point a
candidate of every query, and the codes set the Hamming distances.  What one
query leaves behind must not change what the next one of its tile keeps."""
import numpy as np
import pytest

import oracle
from paper_1805_08995_amd import binding, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _say(msg):
    print(msg, flush=True)


def _codes(rng, base, distances):
    """One code per distance, that many bits of `base` flipped."""
    out = np.empty((len(distances), 2), np.uint64)
    for i, d in enumerate(distances):
        bits = np.zeros(128, np.uint8)
        bits[rng.permutation(128)[:d]] = 1
        out[i] = base ^ np.packbits(bits, bitorder="little").view(np.uint64)
    return out


def _check(images, codes, keys, pairs, tag, band=False, **kw):
    exp = oracle.match_pairs(images, codes, keys, pairs, **kw)
    dev = [torch.from_numpy(im).cuda() for im in images]
    dc = [torch.from_numpy(c.view(np.int64)).cuda() for c in codes]
    dk = [torch.from_numpy(k).cuda() for k in keys]
    for mode in ("batched", "plain"):
        _say(f"{tag} {mode}")
        m = binding.Matcher(mode=mode, k=kw["k"], max_hamming=kw["tau"])
        got, _ = m.match_pairs(dev, dc, dk, pairs)
        for g, e, name in zip(got, exp, ("match_idx", "d1sq", "d2sq")):
            assert np.array_equal(g.cpu().numpy(), e), f"{tag} {mode}: {name}"
        if band:  # a band wider than the images: the same candidates
            kp = [torch.rand(len(im), 2, device="cuda") * 1000 for im in images]
            F = np.tile(np.array([0.0, 0, 0, 0, 0, -1, 0, 1, 0]), (len(pairs), 1))
            got, _ = m.match_pairs_epipolar(dev, dc, dk, kp, pairs, F, 1e5)
            for g, e, name in zip(got, exp, ("match_idx", "d1sq", "d2sq")):
                assert np.array_equal(g.cpu().numpy(), e), f"{tag} {mode} band: {name}"
        m.close()


@pytest.mark.parametrize("tau", [0, 1, 2, 3, 4, 5])
@pytest.mark.parametrize("k", [1, 10, 64])
def test_limit_holds_after_a_crowded_query(tau, k):
    """Queries with 65 to 300 candidates at distance 0, each followed by one with
    fewer than k inside the limit and others just outside it."""
    rng = np.random.default_rng(100 * tau + k)
    a, b = np.zeros(2, np.uint64), np.full(2, ~np.uint64(0))
    images, codes, keys, pairs = [], [], [], []
    nq = 64
    images.append(synth.desc(rng, nq))
    codes.append(np.stack([a, b] * (nq // 2)))
    keys.append(np.zeros((nq, 6), np.uint8))
    for copies in (65, 100, 192, 193, 300):
        near = np.concatenate([np.zeros(min(k, 8) - 1, int), np.repeat([1, 2, 3, 4, 5, 6], 30)])
        tc = np.concatenate([_codes(rng, a, [0] * copies), _codes(rng, b, near)])
        perm = rng.permutation(len(tc))
        pairs.append((0, len(images)))
        images.append(synth.desc(rng, len(tc)))
        codes.append(np.ascontiguousarray(tc[perm]))
        keys.append(np.zeros((len(tc), 6), np.uint8))
    _check(images, codes, keys, np.array(pairs, np.int32), f"tau={tau} k={k}", k=k, tau=tau)


@pytest.mark.parametrize("k", [1, 10, 40, 64])
@pytest.mark.parametrize("tau", [128, 40])
@pytest.mark.parametrize("order", ["nearer", "farther", "equal", "mixed"])
def test_more_candidates_than_the_list_holds(k, tau, order):
    """Around and past the 192 and 256 keys of the list, with the distances
    falling, rising or equal along the index, or crowded at two of them, in the
    plain form and in a band that holds them all."""
    rng = np.random.default_rng(1000 + k)
    a = rng.integers(0, 1 << 63, 2).astype(np.uint64)
    nq = 40
    images, codes, keys = [synth.desc(rng, nq)], [_codes(rng, a, [0, 1, 64] * 13 + [2])], [np.zeros((nq, 6), np.uint8)]
    pairs = []
    for n in (64, 65, 191, 192, 193, 255, 256, 257, 321, 700, 3000):
        d = {"nearer": np.linspace(60, 0, n).astype(int), "farther": np.linspace(0, 60, n).astype(int),
             "equal": np.full(n, 7), "mixed": rng.choice([3, 30, 31, 60], n)}[order]
        pairs.append((0, len(images)))
        images.append(synth.desc(rng, n))
        codes.append(_codes(rng, a, d))
        keys.append(np.zeros((n, 6), np.uint8))
    _check(images, codes, keys, np.array(pairs, np.int32), f"{order} k={k} tau={tau}", band=True, k=k, tau=tau)
