"""Find Peaks with a host count at the limits of the rules that choose between its
short list, its parallel settling and its sorted walk."""
import time

import numpy as np
import pytest

from gpu_common import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    require_gpu()
    from paper_2408_02398_amd import ttm
    return ttm


@pytest.fixture(scope="module")
def ctx(T):
    return T.Context(0)


def _greedy(score, lo, hi, top, dist):
    """The first maximum of the valid box outside the balls of the peaks kept so
    far, again and again (np.argmax takes the lowest index on ties)."""
    s = score[tuple(slice(a, b + 1) for a, b in zip(lo, hi))]
    m = np.where(s > 0, s, np.float32(0.0))
    rows = m.reshape(-1, m.shape[2])
    best = rows.max(axis=1)
    r = int(np.ceil(dist))
    out = []
    while len(out) < top:
        i = int(np.argmax(best))
        if best[i] < 0:
            break
        p = (i // m.shape[1], i % m.shape[1], int(np.argmax(rows[i])))
        out.append([a + b for a, b in zip(p, lo)])
        near = tuple(slice(max(a - r, 0), min(a + r + 1, n)) for a, n in zip(p, m.shape))
        g = np.ogrid[near]
        ball = sum((x.astype(np.int64) - a) ** 2 for x, a in zip(g, p)) < dist * dist
        m[near] = np.where(ball, np.float32(-1.0), m[near])
        m[p] = -1.0
        best.reshape(m.shape[:2])[near[:2]] = m[near[:2]].max(axis=2)
    return out


def _smooth(shape, sigma, seed):
    from scipy.ndimage import gaussian_filter
    a = gaussian_filter(np.random.default_rng(seed).standard_normal(shape).astype(np.float32), sigma)
    return (a - a.min()).astype(np.float32)


def _map(kind, shape):
    rng = np.random.default_rng(sum(shape))
    z, y, x = np.ogrid[:shape[0], :shape[1], :shape[2]]
    if kind == "noise":
        return rng.uniform(0.1, 0.2, shape).astype(np.float32)
    if kind == "smooth":
        return _smooth(shape, 7.0, 3)
    if kind == "plane":        # constant along z and y
        return np.broadcast_to(np.linspace(1, 2, shape[2], dtype=np.float32), shape).copy()
    if kind == "ramp":         # every score in one binade
        return (0.5 + 0.49 * (x + 1.7 * y + 2.3 * z) / sum(k * n for k, n in zip((2.3, 1.7, 1.0), shape))).astype(np.float32)
    if kind == "ramp4":        # scores over four binades
        return (0.2 + 3.0 * (x + 1.7 * y + 2.3 * z) / sum(k * n for k, n in zip((2.3, 1.7, 1.0), shape))).astype(np.float32)
    if kind == "ridges":       # lines falling along x
        s = np.full(shape, 0.1, np.float32) + 1e-4 * rng.random(shape, dtype=np.float32)
        s[5::12, 5::12, :] = np.linspace(2, 1, shape[2], dtype=np.float32)
        return s
    if kind == "constant":
        return np.full(shape, 0.25, np.float32)
    if kind == "checkers":     # every second voxel above its six neighbours
        return (0.5 * ((z + y + x) % 2) + 0.1 * rng.random(shape)).astype(np.float32)
    # maxima only in the blocks of 32 rows that a threshold sampled from every second
    # one reads (even) or leaves out (odd), on noise
    s = 0.1 * rng.random(shape, dtype=np.float32)
    b = np.exp(-((np.arange(-12, 13) ** 2)[:, None, None] + (np.arange(-12, 13) ** 2)[None, :, None] +
                 (np.arange(-12, 13) ** 2)[None, None, :]) / 60.0).astype(np.float32)
    odd = 1 if kind == "unread" else 0
    for i in range(24 if odd else 3):
        zc, yc, xc = 14 + 2 * (i % 6), 64 * (i // 6) + 32 * odd + 16, 20 + 20 * i
        s[zc - 12:zc + 13, yc - 12:yc + 13, xc - 12:xc + 13] += (0.5 + 0.01 * i) * b
    par = (np.arange(shape[1])[None, :, None] // 32 + 5 * np.arange(shape[0])[:, None, None]) % 2
    return np.where((par == odd) | (s < 0.1), s, np.float32(0.05)).astype(np.float32)


@pytest.mark.parametrize("kind,shape,top,dist", [
    ("noise", (50, 60, 70), 1, 9.0),
    ("noise", (50, 60, 70), 16, 9.0),        # the most peaks of the short list
    ("noise", (50, 60, 70), 17, 9.0),        # one more
    ("noise", (16, 17, 30), 8, 5.0),         # 8160 voxels, all in the short list
    ("noise", (16, 17, 31), 8, 5.0),         # 8432: more than it holds
    ("smooth", (64, 64, 64), 16, 14.0),      # the short list holds too few: sorted walk
    ("smooth", (96, 96, 96), 300, 14.0),     # a first list that does not settle, later ones filtered by their leaders
    ("smooth", (96, 90, 100), 1100, 6.0),    # a list of 70 400 that does not settle: the walk of what is left
    ("constant", (30, 40, 50), 12, 9.0),     # equal scores: a longer list than asked for
    ("constant", (60, 70, 70), 1200, 8.0),   # 294 000 candidates in chains
    ("plane", (16, 20, 300), 60, 7.0),
    ("ramp", (44, 50, 60), 1100, 5.0),       # one highest byte: a sorting pass less
    ("ramp4", (44, 50, 60), 1100, 5.0),
    ("ridges", (60, 60, 200), 1500, 5.0),
    ("checkers", (32, 32, 33), 2048, 1.3),   # more kept candidates than are ranked in parallel
    ("read", (40, 512, 512), 100, 12.0),      # a sampled threshold that leaves too few candidates
    ("unread", (40, 512, 512), 100, 12.0),    # and one that leaves many more than asked for
])
def test_find_peaks_routes(T, ctx, kind, shape, top, dist):
    """Positions and values by the rule's definition, bit for bit."""
    import torch
    s = _map(kind, shape)
    lo, hi = (0, 0, 0), tuple(d - 1 for d in shape)
    peaks, vals = T.find_peaks(ctx, torch.from_numpy(s).cuda(), lo, hi, top, dist)
    ref = _greedy(s, lo, hi, top, dist)
    assert peaks.cpu().numpy().tolist() == ref
    assert np.array_equal(vals.cpu().numpy(), np.array([s[tuple(p)] for p in ref], np.float32))


@pytest.mark.parametrize("kind,shape,top,dist", [
    ("plane", (16, 20, 400), 60, 7.0),
    ("constant", (64, 64, 64), 2000, 4.0),
])
def test_chains_cost_no_more_than_the_whole_sort(T, ctx, kind, shape, top, dist):
    """Candidates that wait for each other one after another must not cost more than
    three times the search that sorts every voxel and walks them."""
    import torch
    s = torch.from_numpy(_map(kind, shape)).cuda()
    lo, hi = (0, 0, 0), tuple(d - 1 for d in shape)
    ws = torch.empty(T.load().ttm_workspace_size(T.C.byref(T.make_desc(2, 4, 1.0)), 4, 32, *shape), dtype=torch.uint8,
                     device="cuda")
    p = torch.empty((top, 3), dtype=torch.int32, device="cuda")
    v, n = torch.empty(top, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")

    def best(f):
        t = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            f()
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t)

    whole = best(lambda: T.find_peaks_async(ctx, s, lo, hi, top, dist, p, v, n, ws))
    assert best(lambda: T.find_peaks(ctx, s, lo, hi, top, dist, ws=ws)) <= 3.0 * whole
