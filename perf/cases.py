"""Workloads of the matching path: what a program that uses the library has it do.

Each case names one public entry point of ``binding.Matcher`` (its ``path``) and
the sizes and options of one call:

  codes        hash codes and keys of an image set (device memory)
  match        plain matching of a pair list (device memory)
  noalloc      plain matching in the static device scratch
  epipolar     matching inside a band around known epipolar lines
  fundamental  per-pair fundamental matrices from given matches
  geometric    two-stage matching (subset, estimated matrices, guided stage)
  host         plain matching of host buffers, streamed by the library

Inputs are made on the GPU from a seed, with the statistics of the set-up in
``synth``: SIFT-like uint8 descriptors, scenes whose images share noisy copies
of common points, cameras on an orbit around a cube of 3-D points.  A program
keeps one Matcher per configuration for its whole life; so does this module.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1805_08995_amd import binding, synth

DIM, KEYS, TABLES, ROWS = 128, 256, 6, 176
WIDTH, HEIGHT, FOCAL, ORBIT = 1920, 1080, 1500.0, 500  # the cameras: 500 places on a 40 m circle


def listed():
    return [
        # hashing: the two images of a single match request, where launches count
        {"name": "codes_pair_2000", "path": "codes", "images": 2, "features": 2000},
        # hashing a whole collection at the size of the paper's sets (7.4k-8.6k features per image)
        {"name": "codes_100x8000", "path": "codes", "images": 100, "features": 8000},
        # one image against another: an interactive request
        {"name": "match_pair_2000", "path": "match", "images": 2, "features": 2000},
        # exhaustive matching of a collection, all 4950 pairs (the headline workload)
        {"name": "match_100x8000", "path": "match", "images": 100, "features": 8000},
        # a neighbour list over images of very different sizes (1000-20000 features, 30 partners each)
        {"name": "match_uneven_100", "path": "match", "images": 100, "features": 1000, "features_max": 20000,
         "partners": 30},
        # few images of many features: high-resolution photographs
        {"name": "match_16x20000", "path": "match", "images": 16, "features": 20000},
        # a longer candidate list under a Hamming threshold, on an odd size
        {"name": "match_20x7001_k20_tau48", "path": "match", "images": 20, "features": 7001, "k": 20, "tau": 48},
        # a serving loop that must not allocate: one query image against eight others
        {"name": "noalloc_1x8_3001", "path": "noalloc", "images": 9, "features": 3001},
        # guided matching with known geometry: a stretch of a camera orbit, 30 neighbours each
        {"name": "epipolar_60x12000", "path": "epipolar", "images": 60, "features": 12000, "partners": 30},
        # robust estimation alone, on matches of top-scale subsets
        {"name": "fundamental_600x400", "path": "fundamental", "pairs": 600, "matches": 400},
        # the two-stage form: two scenes, two thirds of the pairs of one scene
        {"name": "geometric_48x12000", "path": "geometric", "images": 48, "features": 12000, "partners": 20,
         "far": 10},
        # a collection in host memory
        {"name": "host_30x8000", "path": "host", "images": 30, "features": 8000},
    ]


def draw(rng):
    def size(lo, hi):  # spread over the logarithm; odd as often as even
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    path = rng.choice(["codes", "match", "match", "match", "noalloc", "epipolar", "fundamental", "geometric", "host"])
    if path == "codes":
        n = size(500, 20000)
        return {"path": path, "images": size(2, max(2, 800000 // n)), "features": n}
    if path == "match":
        n = size(500, 20000)
        c = {"path": path, "images": size(2, max(3, min(100, 300000 // n))), "features": n}
        if rng.random() < 0.3:
            c["features_max"] = min(20000, size(n, 20 * n))
            c["images"], c["partners"] = min(c["images"], 60), size(1, 30)
        if rng.random() < 0.4:
            c["k"], c["tau"] = size(2, 40), rng.choice([128, 64, 48])
        return c
    if path == "noalloc":
        return {"path": path, "images": size(2, 12), "features": size(300, 5000)}
    if path == "epipolar":
        return {"path": path, "images": size(2, 50), "features": size(1000, 12000), "partners": 2 * size(1, 15)}
    if path == "fundamental":
        return {"path": path, "pairs": size(1, 600), "matches": size(16, 800)}
    if path == "geometric":
        return {"path": path, "images": 2 * size(4, 22), "features": size(2000, 12000), "partners": 2 * size(1, 10),
                "far": size(1, 4)}
    return {"path": path, "images": size(2, 25), "features": size(500, 10000)}


# ------------------------------------------------------------------ inputs
_matchers = {}


def matcher(k=10, tau=128, mem="device"):
    """The program's Matcher of this configuration."""
    if (k, tau, mem) not in _matchers:
        _matchers[k, tau, mem] = binding.Matcher(k=k, max_hamming=tau, mem=mem)
    return _matchers[k, tau, mem]


def generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) + 1)


def descriptors(g, n):
    """n SIFT-like descriptors, float32 before rounding to bytes."""
    z = torch.randn(n, DIM, device="cuda", generator=g).abs_()
    z = (z / z.norm(dim=1, keepdim=True)).clamp_(max=0.2)
    return (z / z.norm(dim=1, keepdim=True)).mul_(512.0).round_().clamp_(0, 255)


def noisy(g, x):
    return (x + 8.0 * torch.randn(x.shape, device="cuda", generator=g)).round_().clamp_(0, 255).to(torch.uint8)


def counts_of(case):
    """Features of each image: all equal, or log-uniform up to features_max (the same for every seed)."""
    n, hi = case["features"], case.get("features_max", 0)
    if not hi:
        return [n] * case["images"]
    u = np.random.default_rng(n + hi).uniform(math.log(n), math.log(hi), case["images"])
    return [int(v) for v in np.floor(np.exp(u))]


def scene_images(g, counts):
    """Images of which every tenth sees the same scene: half of an image's
    descriptors are noisy copies from its scene's pool, the rest its own."""
    scenes = min(10, max(1, len(counts) // 2))
    pools = [descriptors(g, 2 * max(counts[s::scenes])) for s in range(scenes)]
    images = []
    for i, n in enumerate(counts):
        pool = pools[i % scenes]
        pick = torch.randperm(len(pool), device="cuda", generator=g)[: n // 2]
        own = descriptors(g, n - n // 2).to(torch.uint8)
        im = torch.cat([noisy(g, pool[pick]), own])
        images.append(im[torch.randperm(n, device="cuda", generator=g)].contiguous())
    return images


def pair_list(case, seed):
    m = case["images"]
    if case["path"] == "noalloc":
        return np.array([(0, j) for j in range(1, m)], np.int32)
    if "partners" not in case:
        return synth.exhaustive_pairs(m)
    rng, out = np.random.default_rng(seed + 1), []
    for i in range(m):
        others = np.delete(np.arange(m), i)
        out += [(i, int(j)) for j in rng.choice(others, size=min(case["partners"], m - 1), replace=False)]
    return np.array(out, np.int32)


def camera(place):
    """Rotation and translation of the camera at this place of the orbit."""
    th = 2.0 * math.pi * place / ORBIT
    c = np.array([40.0 * math.cos(th), 40.0 * math.sin(th), 0.0])
    fwd = -c / np.linalg.norm(c)
    right = np.cross(fwd, [0.0, 0.0, 1.0])
    right /= np.linalg.norm(right)
    R = np.stack([right, np.cross(fwd, right), fwd])
    return R, -R @ c


INTRINSICS = np.array([[FOCAL, 0.0, WIDTH / 2], [0.0, FOCAL, HEIGHT / 2], [0.0, 0.0, 1.0]])


def true_F(a, b):
    """Fundamental matrix of (query place a, train place b)."""
    (Ra, ta), (Rb, tb) = camera(a), camera(b)
    R = Rb @ Ra.T
    t = tb - R @ ta
    skew = np.array([[0.0, -t[2], t[1]], [t[2], 0.0, -t[0]], [-t[1], t[0], 0.0]])
    ki = np.linalg.inv(INTRINSICS)
    return (ki.T @ skew @ R @ ki).reshape(9)


def project(pts, place):
    """Pixel coordinates and depths of the points seen from this place."""
    R, t = camera(place)
    cam = pts @ torch.from_numpy(R.T.copy()).cuda() + torch.from_numpy(t).cuda()
    uvw = cam @ torch.from_numpy(INTRINSICS.T.copy()).cuda()
    return uvw[:, :2] / uvw[:, 2:], cam[:, 2]


def orbit_images(g, n_cams, n_feat, n_points=200_000):
    """Images of one scene from consecutive places of the orbit: keypoints with
    half a pixel of noise, noisy descriptors, feature scales by size and depth."""
    pts = torch.rand(n_points, 3, device="cuda", dtype=torch.float64, generator=g) * 20.0 - 10.0
    base = descriptors(g, n_points)
    size = 0.04 * torch.exp(0.6 * torch.randn(n_points, device="cuda", dtype=torch.float64, generator=g))
    images, kps, scales = [], [], []
    for i in range(n_cams):
        uv, depth = project(pts, i)
        seen = (uv[:, 0] >= 0) & (uv[:, 0] < WIDTH) & (uv[:, 1] >= 0) & (uv[:, 1] < HEIGHT)
        order = torch.rand(n_points, device="cuda", generator=g) + (~seen).float()
        pick = torch.topk(order, n_feat, largest=False).indices
        noise = 0.5 * torch.randn(n_feat, 2, device="cuda", dtype=torch.float64, generator=g)
        jitter = torch.exp(0.1 * torch.randn(n_feat, device="cuda", dtype=torch.float64, generator=g))
        images.append(noisy(g, base[pick]))
        kps.append((uv[pick] + noise).float().contiguous())
        scales.append((FOCAL * size[pick] / depth[pick] * jitter).float().contiguous())
    return images, kps, scales


def near_pairs(n, partners):
    """Each camera with its neighbours on the stretch of the orbit."""
    half = max(1, partners // 2)
    return [(i, j) for i in range(n) for j in range(max(0, i - half), min(n, i + half + 1)) if j != i]


def outputs(n):
    return tuple(torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(3))


def matches_of(case, seed):
    """Planted matches of `fundamental`: per pair, four fifths are noisy
    projections of common points, the rest unrelated; every query point is
    matched, as the slots of a matching call would hold."""
    P, n = case["pairs"], case["matches"]
    g = generator(seed)
    rng = np.random.default_rng(seed)
    kps, pairs, idx = [], [], []
    for p in range(P):
        a = int(rng.integers(0, ORBIT))
        b = a + int(rng.integers(4, 30))
        pts = torch.rand(n, 3, device="cuda", dtype=torch.float64, generator=g) * 20.0 - 10.0
        perm = torch.randperm(n, device="cuda", generator=g)
        q, t = project(pts, a)[0], project(pts, b)[0]
        t[: n // 5] = torch.rand(n // 5, 2, device="cuda", dtype=torch.float64, generator=g) * float(HEIGHT)
        noise = 0.5 * torch.randn(2, n, 2, device="cuda", dtype=torch.float64, generator=g)
        kps += [(q + noise[0]).float().contiguous(), (t + noise[1]).float()[perm].contiguous()]
        idx.append(torch.argsort(perm).int())
        pairs.append((2 * p, 2 * p + 1))
    return kps, np.array(pairs, np.int32), torch.cat(idx)


def prepare(case, seed):
    path = case["path"]
    g = generator(seed)
    m = matcher(case.get("k", 10), case.get("tau", 128), "host" if path == "host" else "device")
    s = {"path": path, "m": m}
    rand8 = np.random.default_rng(seed + 7).integers(0, 1 << 32, (256, 8), dtype=np.uint64).astype(np.uint32)
    if path == "fundamental":
        kps, s["pairs"], s["idx"] = matches_of(case, seed)
        s["n_feat"] = np.full(len(kps), case["matches"], np.int32)
        s["kps"], s["rand8"] = m.bind(kps), rand8
        return s
    if path == "epipolar":
        images, kps, _ = orbit_images(g, case["images"], case["features"])
        s["pairs"] = np.array(near_pairs(case["images"], case["partners"]), np.int32)
        s["F"] = np.array([true_F(a, b) for a, b in s["pairs"]])
        s["kps"] = m.bind(kps)
    elif path == "geometric":
        half = case["images"] // 2
        a, b = orbit_images(g, half, case["features"]), orbit_images(g, half, case["features"])
        images, kps, scales = (x + y for x, y in zip(a, b))
        near = near_pairs(half, case["partners"])
        rng = np.random.default_rng(seed + 2)
        far = [(i, int(j) + (half if i < half else 0)) for i in range(2 * half)
               for j in rng.choice(half, size=min(half, case["far"]), replace=False)]
        s["pairs"] = np.array(near + [(i + half, j + half) for i, j in near] + far, np.int32)
        s["kps"], s["scales"], s["rand8"] = m.bind(kps), m.bind(scales), rand8
    else:
        images = scene_images(g, counts_of(case))
        s["pairs"] = pair_list(case, seed)
    dev = m if path != "host" else matcher()
    # the codes and keys of the set's images lie one after another
    n_feat = [int(im.shape[0]) for im in images]
    s["all_codes"] = torch.zeros(sum(n_feat), 2, dtype=torch.int64, device="cuda")
    s["all_keys"] = torch.zeros(sum(n_feat), TABLES, dtype=torch.uint8, device="cuda")
    codes, keys = list(s["all_codes"].split(n_feat)), list(s["all_keys"].split(n_feat))
    if path != "codes":
        dev.build_codes(images, out=(codes, keys))
    n_q = sum(n_feat[q] for q in s["pairs"][:, 0])
    if path == "host":
        to_host = lambda arrs, view: [a.cpu().numpy().view(view) for a in arrs]  # noqa: E731
        images, codes, keys = to_host(images, np.uint8), to_host(codes, np.uint64), to_host(keys, np.uint8)
        s["out"] = tuple(np.zeros(n_q, np.int32) for _ in range(3))
    elif path != "codes":
        s["out"] = outputs(n_q)
    s["images"], s["codes"], s["keys"] = m.bind(images), m.bind(codes), m.bind(keys)
    return s


def run(s):
    m, path = s["m"], s["path"]
    if path == "codes":
        m.build_codes(s["images"], out=(s["codes"], s["keys"]))
        return s["all_codes"], s["all_keys"]
    if path == "fundamental":
        return m.estimate_fundamental(s["n_feat"], s["kps"], s["pairs"], s["idx"], s["rand8"])
    args = s["images"], s["codes"], s["keys"]
    if path == "noalloc":
        return m.match_pairs_noalloc(*args, s["pairs"], s["out"])[0]
    if path == "epipolar":
        return m.match_pairs_epipolar(*args, s["kps"], s["pairs"], s["F"], 4.0, out=s["out"])[0]
    if path == "geometric":
        return m.match_pairs_geometric(*args, s["kps"], s["scales"], s["pairs"], s["rand8"], out=s["out"])[:2]
    return m.match_pairs(*args, s["pairs"], out=s["out"])[0]


# ------------------------------------------------------------------ the work a pass cannot do without
def work(case):
    path = case["path"]
    if path == "fundamental":
        P, n, hyp = case["pairs"], case["matches"], 256
        # eight-point solve and rank 2 per hypothesis, the inlier test of every match, the refit
        return {"bytes": P * (n * 20 + 88), "flops": P * (hyp * (1000 + 20 * n) + 90 * n)}
    lo, hi = case["features"], case.get("features_max", 0)
    n = (hi - lo) / math.log(hi / lo) if hi > lo else lo  # mean features per image
    m = case["images"]
    if path == "codes":
        return {"bytes": m * n * (DIM + 22), "flops": 2 * m * n * DIM * ROWS}
    k = case.get("k", 10)
    # per query: 128-bit Hamming distances of its bucket entries (8 operations on words each), k exact distances
    plain = lambda t: TABLES * t / KEYS * 8 + k * 3 * DIM  # noqa: E731
    band = lambda t: TABLES * t / KEYS * 7 + k * 3 * DIM  # noqa: E731
    if path == "geometric":
        near = 2 * len(near_pairs(m // 2, case["partners"]))
        far = m * min(m // 2, case["far"])
        ops = (near + far) * (n / 5) * plain(n / 5) + near * (256 * (1000 + 20 * n / 20) + n * band(n))
        return {"bytes": m * n * (DIM + 22 + 12) + (near + far) * n * 12, "flops": ops}
    if path == "epipolar":
        P = len(near_pairs(m, case["partners"]))
        return {"bytes": m * n * (DIM + 22 + 8) + P * (n * 12 + 72), "flops": P * n * band(n)}
    P = m - 1 if path == "noalloc" else m * min(case["partners"], m - 1) if "partners" in case else m * (m - 1) // 2
    return {"bytes": m * n * (DIM + 22) + P * n * 12, "flops": P * n * plain(n)}


# ------------------------------------------------------------------ reference in 64 bits
def rank2(F):
    """F [.., 3, 3] without its component along the smallest eigenvector of F^T F."""
    v = np.linalg.eigh(np.swapaxes(F, -1, -2) @ F)[1][..., :, :1]
    return F - (F @ v) @ np.swapaxes(v, -1, -2)


def smallest_eigenvector(A):
    """Cyclic Jacobi on a symmetric 9 x 9 matrix, with the signs that rotations from the identity give."""
    A, V = A.copy(), np.eye(9)
    for _ in range(10):
        for p in range(8):
            for q in range(p + 1, 9):
                if A[p, q] == 0.0:
                    continue
                theta = (A[q, q] - A[p, p]) / (2.0 * A[p, q])
                t = (-1.0 if theta < 0 else 1.0) / (abs(theta) + math.sqrt(theta * theta + 1.0))
                c = 1.0 / math.sqrt(t * t + 1.0)
                J = np.array([[c, t * c], [-t * c, c]])
                A[:, [p, q]] = A[:, [p, q]] @ J
                A[[p, q]] = J.T @ A[[p, q]]
                V[:, [p, q]] = V[:, [p, q]] @ J
    return V[:, np.argmin(np.diag(A))]


def inliers(F, q, t, px):
    line = q @ np.swapaxes(F, -1, -2)
    e = (line * t).sum(-1)
    return e * e <= px * px * (line[..., 0] ** 2 + line[..., 1] ** 2)


def estimate(q, t, rand8, px=2.0):
    """The fundamental matrix of matches q <-> t ([n, 3], homogeneous)."""
    n, T = len(q), []
    for x in (q, t):
        c = x[:, :2].mean(0)
        s = math.sqrt(2.0) / np.linalg.norm(x[:, :2] - c, axis=1).mean()
        T.append(np.array([[s, 0, -s * c[0]], [0, s, -s * c[1]], [0, 0, 1]]))
    a = np.einsum("ni,nj->nij", t @ T[1].T, q @ T[0].T).reshape(n, 9)
    sample = np.zeros(rand8.shape, np.int64)
    for i in range(8):  # eight distinct matches per hypothesis
        j = n - 8 + i
        v = (rand8[:, i].astype(np.uint64) * np.uint64(j + 1) >> np.uint64(32)).astype(np.int64)
        sample[:, i] = np.where((sample[:, :i] == v[:, None]).any(1), j, v)
    A = a[sample]
    f = np.concatenate([np.linalg.solve(A[:, :, :8], -A[:, :, 8:])[..., 0], np.ones((len(A), 1))], 1)
    F = T[1].T @ rank2(f.reshape(-1, 3, 3)) @ T[0]
    best = inliers(F, q, t, px).sum(1).argmax()
    keep = a[inliers(F[best], q, t, px)]
    return (T[1].T @ rank2(smallest_eigenvector(keep.T @ keep).reshape(3, 3)) @ T[0]).reshape(9)


def exact(case, seed):
    """F of `fundamental`; every other output is a whole number, and the two-stage form's matrices follow from
    a matching stage that takes too long here."""
    if case["path"] != "fundamental":
        return None
    kps, pairs, idx = matches_of(case, seed)
    rand8 = np.random.default_rng(seed + 7).integers(0, 1 << 32, (256, 8), dtype=np.uint64).astype(np.uint32)
    idx = idx.cpu().numpy().reshape(len(pairs), -1)
    one = lambda x: np.concatenate([x.cpu().numpy().astype(np.float64), np.ones((len(x), 1))], 1)  # noqa: E731
    F = np.array([estimate(one(kps[a]), one(kps[b])[idx[p]], rand8) for p, (a, b) in enumerate(pairs)])
    return {"F": F, "n_matches": None, "n_inliers": None, "best_h": None, "status": None}
