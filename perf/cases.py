"""Timed work of the framework: what a program that uses it has it do, from the
smallest call to a 512^3 tile, through the public entry points of
paper_2408_02398_amd.ttm.

A case is a dict of plain values.  Its `kind` names the path:

  pass      a whole small tomogram: Engine.run with the 16-start orientation
            and Find Peaks (a 64^3 box at degree 4: launches and latency count)
  item      one subtomogram of a batch: normalize, then correlate
  tile      one FFT tile of a big tomogram: normalize_correlate (degree 6;
            256^3 and 512^3 tiles)
  localise  the quaternion form: a score-only Engine pass, Find Peaks, then
            TTM-ref around every peak
  batch     uneven subtomograms of two templates in one HIP graph
            (BatchEngine, learned start)
  extract   score and orientation of a field box, from 16 fixed starts or from
            the learned start with the multistart fallback
  peaks     Find Peaks over a whole score map
  train     one training step of the learned start's network
  template  the tensor template of a density (Alg. 1)

Inputs: Gaussian-blob densities, copies of them in random rotations on a
jittered lattice, white noise at a stated SNR, optionally without the +-60
degree missing wedge.  Tensor templates, fields and networks that a case needs
as inputs are made with torch in 64 bits, so they do not depend on the code
under test.
"""
import itertools
import math

import numpy as np
import torch

from paper_2408_02398_amd import ttm

DEV = "cuda"
F64 = torch.float64
_kept = {}     # context, templates and networks that a program keeps for its whole life


# ----------------------------------------------------------------------------
# cases
# ----------------------------------------------------------------------------

def listed():
    return [
        # the smallest whole pass: one 64^3 box, its five best peaks
        dict(name="pass_64_n4", kind="pass", nz=64, ny=64, nx=64, n=4, L=16, r=7.0, N=64, top=5),
        # the smallest subtomogram of the batch workload
        dict(name="item_96_n6", kind="item", nz=96, ny=96, nx=96, n=6, L=24, r=10.0, N=96, bf16=False),
        # a ragged subtomogram over several 128^3 tiles, field stored as bfloat16
        dict(name="item_ragged_bf16", kind="item", nz=150, ny=171, nx=190, n=6, L=32, r=14.0, N=128, bf16=True),
        # a 256^3 tile: the middle workload's whole volume
        dict(name="tile_256_n6", kind="tile", N=256, n=6, L=32, r=14.0, bf16=False),
        # a 512^3 tile of the large tomogram: the largest call
        dict(name="tile_512_n6", kind="tile", N=512, n=6, L=40, r=17.0, bf16=False),
        # position search and refinement in the quaternion form: 125 copies in 197^3
        dict(name="localise_197_q4", kind="localise", grid=5, spacing=40, L=32, r=14.0, n=4, N=256, snr=3.0),
        # four uneven subtomograms of two templates in one graph launch
        dict(name="batch_learned", kind="batch", edges="96,128,160,128", n=6, top=30),
        # the learned orientation of every voxel of a 256^3 tile
        dict(name="extract_learned_217", kind="extract", bz=217, by=217, bx=217, n=6, L=40, learned=True),
        # the 16-start orientation of a 128^3 tile
        dict(name="extract_plain_97", kind="extract", bz=97, by=97, bx=97, n=6, L=32, learned=False),
        # the large tomogram's score map, 2000 peaks
        dict(name="peaks_512x928", kind="peaks", nz=512, ny=928, nx=928, r=17.0, L=40, top=2000),
        # one step of the network's training at its usual batch
        dict(name="train_8192", kind="train", n=6, B=8192),
        # the large workload's tensor template: 24 000 rotations of a 40^3 box
        dict(name="template_40_24000", kind="template", L=40, r=17.0, n=6, dprime=3, nq=24000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["pass", "item", "item", "tile", "localise", "extract", "extract", "peaks",
                       "train", "template"])
    if kind == "pass":
        L = rng.choice([8, 11, 12, 16])
        nz, ny, nx = (rng.randint(36, 72) for _ in range(3))
        return dict(kind=kind, nz=nz, ny=ny, nx=nx, n=rng.choice([2, 4]), L=L, r=L / 2 - 1.0,
                    N=rng.choice([32, 64]), top=rng.randint(2, 8))
    if kind == "item":
        L = rng.choice([24, 27, 32, 40])
        nz, ny, nx = (_log(rng, 64, 220) for _ in range(3))
        return dict(kind=kind, nz=nz, ny=ny, nx=nx, n=rng.choice([4, 6]), L=L, r=0.43 * L,
                    N=rng.choice([64, 96, 128, 160, 192]), bf16=rng.random() < 0.3)
    if kind == "tile":
        L = rng.choice([24, 32, 33, 40, 48])
        return dict(kind=kind, N=rng.choice([128, 160, 192, 256, 256]), n=rng.choice([2, 4, 6]), L=L,
                    r=0.43 * L, bf16=rng.random() < 0.3)
    if kind == "localise":
        return dict(kind=kind, grid=rng.randint(2, 4), spacing=rng.randint(36, 44), L=rng.choice([27, 32]),
                    r=rng.choice([12.0, 13.0]), n=rng.choice([2, 4]), N=rng.choice([128, 192, 256]),
                    snr=rng.choice([3.0, 10.0]))
    if kind == "extract":
        learned = rng.random() < 0.6
        e = [_log(rng, 24, 200 if learned else 100) for _ in range(3)]
        return dict(kind=kind, bz=e[0], by=e[1], bx=e[2], n=rng.choice([4, 6]), L=rng.choice([32, 40]),
                    learned=learned)
    if kind == "peaks":
        e = [_log(rng, 64, 700) for _ in range(3)]
        L = rng.choice([24, 32, 40])
        if math.prod(v // (2 * int(0.43 * L)) + 1 for v in e) > 16384:
            L = 40        # the peak search's grid of 2r cells holds at most 16384
        r = float(int(0.43 * L))
        room = 1.0
        for v in e:
            room *= max(1, (v - L + 1) // (L + 4))
        return dict(kind=kind, nz=e[0], ny=e[1], nx=e[2], r=r, L=L, top=max(1, min(2000, int(room * 0.8))))
    if kind == "train":
        return dict(kind=kind, n=rng.choice([2, 4, 6]), B=_log(rng, 1024, 16384))
    L = rng.choice([16, 24, 31, 32, 40])
    return dict(kind=kind, L=L, r=0.43 * L, n=rng.choice([2, 4, 6]), dprime=rng.choice([3, 3, 4]),
                nq=_log(rng, 1200, 24000))


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _kept_once(key, make):
    if key not in _kept:
        _kept[key] = make()
    return _kept[key]


def _ctx():
    return _kept_once("ctx", lambda: ttm.Context(0))


def _exponents(n, d):
    """Component exponents in graded-lex order, and their multinomial weights."""
    ex = [e for e in itertools.product(range(n, -1, -1), repeat=d) if sum(e) == n]
    mu = [math.factorial(n) / math.prod(math.factorial(k) for k in e) for e in ex]
    return ex, torch.tensor(mu, dtype=F64, device=DEV)


def _rot(q):
    """Rotation matrices (..., 3, 3) of unit quaternions (w, x, y, z)."""
    w, x, y, z = (q / q.norm(dim=-1, keepdim=True)).unbind(-1)
    rows = [1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
            2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
            2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]
    return torch.stack(rows, -1).view(*q.shape[:-1], 3, 3)


def _spiral(n):
    """n quaternions of the super-Fibonacci spiral on S^3 (Alexa 2022)."""
    s = torch.arange(n, dtype=F64, device=DEV) + 0.5
    a, b = 2 * math.pi * s / math.sqrt(2.0), 2 * math.pi * s / 1.533751168755204288118041
    r, R = torch.sqrt(s / n), torch.sqrt(1 - s / n)
    return torch.stack([r * torch.sin(a), r * torch.cos(a), R * torch.sin(b), R * torch.cos(b)], 1)


def _starts(count, dim):
    s = np.random.default_rng(7).standard_normal((count, dim))
    s /= np.linalg.norm(s, axis=1, keepdims=True)
    s[s[:, -1 if dim == 3 else 0] < 0] *= -1.0
    return torch.from_numpy(s.astype(np.float32)).to(DEV)


def _points(L):
    """(L^3, 3) points (x, y, z) of the box relative to its centre L // 2."""
    i = torch.arange(L, dtype=F64, device=DEV) - L // 2
    z, y, x = torch.meshgrid(i, i, i, indexing="ij")
    return torch.stack([x, y, z], -1).view(-1, 3)


def _model(seed, blobs=4):
    rng = np.random.default_rng(seed)
    q = torch.from_numpy(rng.standard_normal((blobs, 4))).to(DEV)
    return (torch.from_numpy(rng.uniform(-4, 4, (blobs, 3))).to(DEV), _rot(q),
            torch.from_numpy(rng.uniform(1.5, 3.0, (blobs, 3))).to(DEV))


def _density(model, pts):
    out = 0.0
    for c, axes, sig in zip(*model):
        out = out + torch.exp(-0.5 * (((pts - c) @ axes / sig) ** 2).sum(-1))
    return out


def _ball(L, r):
    return ((_points(L) ** 2).sum(-1) <= float(np.float32(r)) ** 2).to(F64).view(L, L, L)


def _filter(t, axis, a, replicate):
    w = float(np.float32(a))
    n = t.shape[axis]
    lo, hi = t.narrow(axis, 0, n - 1), t.narrow(axis, 1, n - 1)
    edge0, edge1 = t.narrow(axis, 0, 1), t.narrow(axis, n - 1, 1)
    if not replicate:
        edge0, edge1 = torch.zeros_like(edge0), torch.zeros_like(edge1)
    return w * torch.cat([edge0, lo], axis) + (1 - 2 * w) * t + w * torch.cat([hi, edge1], axis)


def _prefilter(t, replicate):
    for axis in range(3):
        t = _filter(t, axis, 0.2, replicate)
    return t


def _normalised(tmpl, L, r):
    """t' of Eq. norm_t."""
    m = _ball(L, r)
    s = m * _prefilter(tmpl.to(F64), False)
    mu = s.sum() / m.sum()
    return m * (s - mu) / torch.sqrt((s * s).sum() - s.sum() ** 2 / m.sum())


def _tensor_template(tmpl, L, r, quats, n, d):
    """(T, t') of Alg. 1 in 64 bits: trilinear pull-backs weighted by v_q^alpha."""
    tn = _normalised(tmpl, L, r)
    P = L + 4
    flat = torch.nn.functional.pad(tn, (2,) * 6).view(-1)
    ex, _ = _exponents(n, d)
    pts = _points(L)
    R = _rot(quats)
    v = (quats / quats.norm(dim=1, keepdim=True)) if d == 4 else R[:, :, 2]
    mono = torch.stack([torch.prod(torch.stack([v[:, i] ** e[i] for i in range(d)]), 0) for e in ex])
    T = torch.zeros((len(ex), L ** 3), dtype=F64, device=DEV)
    for q0 in range(0, len(quats), 64):
        src = (pts @ R[q0:q0 + 64] + L // 2).clamp(-1.5, L + 0.5)     # R^T p, (q, L^3, 3)
        f = torch.floor(src)
        t, i = src - f, f.long() + 2
        val = 0.0
        for dx, dy, dz in itertools.product((0, 1), repeat=3):
            wgt = 1.0
            for k, o in enumerate((dx, dy, dz)):
                wgt = wgt * (t[..., k] if o else 1 - t[..., k])
            val = val + wgt * flat[((i[..., 2] + dz) * P + i[..., 1] + dy) * P + i[..., 0] + dx]
        T += mono[:, q0:q0 + 64] @ val
    return (T / len(quats)).view(-1, L, L, L), tn


def _template(n, L, r, d=3, seed=2):
    """A template's density model, tensor template (float32) and t', kept for the process."""
    def make():
        model = _model(1000 * seed + L)
        T, tn = _tensor_template(_density(model, _points(L)).view(L, L, L), L, r, _spiral(1200), n, d)
        return model, T.float().contiguous(), tn.float().contiguous()
    return _kept_once(("template", n, L, r, d, seed), make)


def _tomogram(shape, model, L, r, snr, seed, spacing=None, jitter=True, wedge=False):
    """float32 volume: rotated copies on a jittered lattice, white noise at `snr`."""
    g = _gen(seed)
    sp = spacing or L + 6
    m0 = L // 2 + 2 if spacing else L // 2
    ax = [torch.arange(m0, max(m0 + 1, s - (L - L // 2)), sp, device=DEV) for s in shape]
    c = torch.stack(torch.meshgrid(*ax, indexing="ij"), -1).view(-1, 3)
    if jitter:
        c = c + torch.randint(0, 5, c.shape, generator=g, device=DEV)
    dims = torch.tensor(shape, device=DEV)
    c = c[((c - L // 2 >= 0) & (c + L - L // 2 <= dims)).all(1)]
    R = _rot(torch.randn((len(c), 4), generator=g, device=DEV, dtype=F64))
    pts = _points(L)
    i = pts.long()
    off = (i[:, 2] * shape[1] + i[:, 1]) * shape[2] + i[:, 0]
    sd = torch.sqrt(_density(model, pts)[_ball(L, r).view(-1) > 0].var() / snr).float()
    vol = torch.randn(shape, generator=g, device=DEV) * sd
    flat = vol.view(-1)
    for k in range(0, len(c), 32):       # the copies' boxes are disjoint
        cc = c[k:k + 32]
        idx = ((cc[:, 0] * shape[1] + cc[:, 1]) * shape[2] + cc[:, 2])[:, None] + off[None]
        flat[idx] += _density(model, pts @ R[k:k + 32]).float()
    if wedge:
        s = torch.fft.rfftn(vol)
        kz = torch.fft.fftfreq(shape[0], device=DEV).abs()[:, None, None]
        kx = torch.fft.rfftfreq(shape[2], device=DEV)[None, None, :]
        s *= kz <= math.tan(math.radians(60.0)) * kx + 1e-12
        vol = torch.fft.irfftn(s, s=shape).contiguous()
    return vol


def _field(vol, T, L, r):
    """(g, w, stats, C) in 64 bits on the whole valid region (w there too), one FFT of the volume's own extent."""
    g = _prefilter(vol.to(F64), True)
    m = _ball(L, r)
    shape = tuple(vol.shape)
    U = tuple(s - L + 1 for s in shape)

    def corr(G, t):
        return torch.fft.irfftn(G * torch.fft.rfftn(t, s=shape).conj(), s=shape)[:U[0], :U[1], :U[2]]

    mean, msq = g.mean(), (g * g).mean()
    gc = g - mean
    s1, s2 = corr(torch.fft.rfftn(gc), m), corr(torch.fft.rfftn(gc * gc), m)
    var = s2 - s1 * s1 / m.sum()
    w = torch.where(var > float(np.float32(1e-6)) * m.sum() * msq, var.clamp_min(1e-300).rsqrt(), torch.zeros_like(var))
    G = torch.fft.rfftn(g)
    C = torch.empty((len(T), *U), dtype=F64, device=DEV)
    for k in range(len(T)):
        C[k] = w * corr(G, T[k].to(F64))
    return g, w, torch.stack([mean, msq]), C


def _score(C, n, d):
    _, mu = _exponents(n, d)
    s = torch.zeros(C.shape[1:], dtype=F64, device=DEV)
    for k in range(len(C)):
        s += mu[k] * C[k].to(F64) ** 2
    return s.sqrt()


def _full(part, shape, L):
    """A valid-region map in a full-size one, 0 outside."""
    out = torch.zeros(shape, dtype=F64, device=DEV)
    c = L // 2
    out[c:c + part.shape[0], c:c + part.shape[1], c:c + part.shape[2]] = part
    return out


def _network(n, L, r, seed=2):
    """Trained network parameters in the framework's layout: W1 [32][64], b1,
    W2 [64][64], b2, W3 [64][16], b3.  Trained with torch to raise <C, u^n> /
    ||C|| at u = net(C) on voxels of one tomogram of the template."""
    def make():
        model, T, _ = _template(n, L, r, 3, seed)
        C = _field(_tomogram((112, 112, 112), model, L, r, 0.1, 91, wedge=False), T, L, r)[3]
        ex, mu = _exponents(n, 3)
        X = (mu.sqrt()[:, None] * C.view(len(ex), -1))
        X = (X / X.norm(dim=0).clamp_min(1e-30)).t().float().contiguous()
        e = torch.tensor(ex, device=DEV)
        rng = np.random.default_rng(5)
        shapes = [(len(ex), 64), (64,), (64, 64), (64,), (64, 3), (3,)]
        p = [torch.from_numpy((rng.standard_normal(s) * math.sqrt(2.0 / s[0]) if len(s) == 2 else np.zeros(s))
                              .astype(np.float32)).to(DEV).requires_grad_() for s in shapes]
        opt = torch.optim.Adam(p, lr=3e-3)
        sq = mu.sqrt().float()
        g = _gen(17)
        steps = 2500
        for k in range(steps):
            x = X[torch.randint(0, len(X), (4096,), generator=g, device=DEV)]
            y = torch.relu(torch.relu(x @ p[0] + p[1]) @ p[2] + p[3]) @ p[4] + p[5]
            u = y / y.norm(dim=1, keepdim=True)
            pw = [torch.ones_like(u)]
            for _ in range(n):
                pw.append(pw[-1] * u)
            pw = torch.stack(pw)                               # [power][sample][axis]
            mono = pw[e[:, 0], :, 0] * pw[e[:, 1], :, 1] * pw[e[:, 2], :, 2]
            loss = -(x * (sq[:, None] * mono).t()).sum(1).mean()
            for group in opt.param_groups:
                group["lr"] = 1e-4 + 1.45e-3 * (1 + math.cos(math.pi * k / steps))
            opt.zero_grad()
            loss.backward()
            opt.step()
        W1, W3, b3 = torch.zeros((32, 64), device=DEV), torch.zeros((64, 16), device=DEV), torch.zeros(16, device=DEV)
        with torch.no_grad():
            W1[:len(ex)], W3[:, :3], b3[:3] = p[0], p[4], p[5]
            return torch.cat([W1.flatten(), p[1], p[2].flatten(), p[3], W3.flatten(), b3]).contiguous()
    return _kept_once(("network", n, L, r, seed), make)


def _shape(case):
    return (case["N"],) * 3 if case["kind"] == "tile" else (case["nz"], case["ny"], case["nx"])


def _volume(case, seed):
    model, T, _ = _template(case["n"], case["L"], case["r"])
    shape = _shape(case)
    kind = case["kind"]
    snr = 2.0 if kind == "pass" else 0.1
    return _tomogram(shape, model, case["L"], case["r"], snr, seed, wedge=kind == "tile"), T


def _grid_volume(case, seed):
    model, T, tn = _template(case["n"], case["L"], case["r"], 4)
    e = 2 * (case["L"] // 2 + 2) + (case["grid"] - 1) * case["spacing"] + 1
    vol = _tomogram((e, e, e), model, case["L"], case["r"], case["snr"], seed, spacing=case["spacing"], jitter=False)
    return vol, T, tn


_BATCH = ((24, 10.0), (32, 14.0))     # the batch's templates: box edge, mask radius


def _batch_volumes(case, seed):
    out = []
    for i, e in enumerate(int(v) for v in case["edges"].split(",")):
        L, r = _BATCH[i % 2]
        out.append(_tomogram((e, e, e), _template(case["n"], L, r)[0], L, r, 0.1, 100 * seed + i))
    return out


def _score_map(case, seed):
    """A score map as ||C||_F of noise looks (narrow, smooth), with `top` and some more peaks."""
    g = _gen(seed)
    shape = _shape(case)
    s = torch.randn(shape, generator=g, device=DEV)
    for axis in range(3):
        s = _filter(s, axis, 0.2, True)
        s = _filter(s, axis, 0.2, True)
    s = (0.03 * s).add_(0.2)
    L = case["L"]
    ax = [torch.arange(L // 2 + 2, v - L // 2 - 3, L + 4, device=DEV) for v in shape]
    c = torch.stack(torch.meshgrid(*ax, indexing="ij"), -1).view(-1, 3)
    c = c + torch.randint(-2, 3, c.shape, generator=g, device=DEV)
    c = c[torch.randperm(len(c), generator=g, device=DEV)[:int(1.2 * case["top"]) + 1]]
    h = 6
    i = torch.arange(-h, h + 1, device=DEV)
    oz, oy, ox = (t.reshape(-1) for t in torch.meshgrid(i, i, i, indexing="ij"))
    bump = torch.exp(-(oz * oz + oy * oy + ox * ox).float() / (2 * 2.5 ** 2))
    high = 0.08 + 0.15 * torch.rand(len(c), generator=g, device=DEV)
    idx = ((c[:, 0] * shape[1] + c[:, 1]) * shape[2] + c[:, 2])[:, None] + ((oz * shape[1] + oy) * shape[2] + ox)[None]
    s.view(-1)[idx] += high[:, None] * bump[None]
    k = L // 2
    out = torch.zeros(shape, device=DEV)
    (z, y, x) = (slice(k, v - L + k + 1) for v in shape)
    out[z, y, x] = s[z, y, x]
    return out


def _pairs(case, seed):
    """Training pairs: noisy rank-one tensors v^n and their axes, batch x K and batch x 3."""
    g = _gen(seed)
    ex, _ = _exponents(case["n"], 3)
    v = torch.randn((case["B"], 3), generator=g, device=DEV, dtype=F64)
    v = v / v.norm(dim=1, keepdim=True)
    mono = torch.stack([v[:, 0] ** e[0] * v[:, 1] ** e[1] * v[:, 2] ** e[2] for e in ex], 1)
    C = mono + 0.15 * torch.randn(mono.shape, generator=g, device=DEV, dtype=F64)
    rng = np.random.default_rng(seed)
    W1, W3 = np.zeros((32, 64)), np.zeros((64, 16))
    W1[:len(ex)] = rng.standard_normal((len(ex), 64)) * math.sqrt(2.0 / len(ex))
    W2 = rng.standard_normal((64, 64)) * math.sqrt(2.0 / 64)
    W3[:, :3] = rng.standard_normal((64, 3)) / 8.0
    z, b = np.zeros(64), np.zeros(16)
    p = np.concatenate([W1.ravel(), z, W2.ravel(), z, W3.ravel(), b]).astype(np.float32)
    return C.float().contiguous(), v.float().contiguous(), torch.from_numpy(p).to(DEV)


def _density_box(case, seed):
    L = case["L"]
    return _density(_model(seed), _points(L)).view(L, L, L).float().contiguous(), _spiral(case["nq"]).float().contiguous()


# ----------------------------------------------------------------------------
# what a program has in hand before the call
# ----------------------------------------------------------------------------

def prepare(case, seed):
    kind, ctx = case["kind"], _ctx()
    s = dict(case=dict(case), ctx=ctx)
    if kind in ("pass", "item", "tile"):
        vol, T = _volume(case, seed)
        d = ttm.make_desc(case["n"], case["L"], case["r"])
        spec = ttm.template_spectra(ctx, d, T, case["N"])
        s.update(vol=vol, desc=d, spec=spec, dtype=torch.bfloat16 if case.get("bf16") else torch.float32)
        lo, hi = ttm.valid_bounds(vol.shape, case["L"])
        s.update(lo=lo, size=tuple(b - a + 1 for a, b in zip(lo, hi)))
        if kind == "pass":
            s["engine"] = ttm.Engine(ctx, d, spec, case["N"], tuple(vol.shape), _starts(16, 3))
        if kind == "tile":
            s["g"], s["w"], s["stats"] = ttm.prefilter(ctx, d, vol)
            K = ttm.n_components(case["n"])
            s["out"] = torch.empty((K, *s["size"]), dtype=s["dtype"], device=DEV)
            s["ws"] = ttm._ws(d, ttm.L.TTM_OP_NORM_CORR, case["N"], device=DEV)
    elif kind == "localise":
        vol, T, tn = _grid_volume(case, seed)
        d = ttm.make_desc(case["n"], case["L"], case["r"], dprime=4)
        spec = ttm.template_spectra(ctx, d, T, case["N"])
        s.update(vol=vol, desc=d, T=T, tn=tn, starts=_starts(32, 4),
                 engine=ttm.Engine(ctx, d, spec, case["N"], tuple(vol.shape), None, orient=False))
    elif kind == "batch":
        vols = _batch_volumes(case, seed)
        descs = [ttm.make_desc(case["n"], L, r) for L, r in _BATCH]
        templates = [(d, _template(case["n"], L, r)[1]) for d, (L, r) in zip(descs, _BATCH)]
        nets = [ttm.MLP(ctx, d, _network(case["n"], L, r)) for d, (L, r) in zip(descs, _BATCH)]
        owner = [i % 2 for i in range(len(vols))]
        be = ttm.BatchEngine(ctx, templates, [tuple(v.shape) for v in vols], owner, _starts(16, 3), case["top"],
                             mlps=nets, kappa=float("-inf"))
        be.capture()
        s.update(vols=vols, engine=be, nets=nets)
    elif kind == "extract":
        n, L = case["n"], case["L"]
        r = float(int(0.43 * L))
        model, T, _ = _template(n, L, r)
        box = (case["bz"], case["by"], case["bx"])
        C = _field(_tomogram(tuple(b + L - 1 for b in box), model, L, r, 0.1, seed), T, L, r)[3].float().contiguous()
        d = ttm.make_desc(n, L, r)
        s.update(C=C, desc=d, starts=_starts(16, 3), ws=ttm._ws(d, ttm.L.TTM_OP_EXTRACT, 0, box, device=DEV),
                 score=torch.zeros(box, device=DEV), lam=torch.zeros(box, device=DEV),
                 dir=torch.zeros((*box, 3), device=DEV), fb=torch.zeros(1, dtype=torch.int32, device=DEV),
                 net=ttm.MLP(ctx, d, _network(n, L, r)) if case["learned"] else None)
    elif kind == "peaks":
        s["score"] = _score_map(case, seed)
        s["ws"] = ttm._ws(ttm.make_desc(2, 4, 1.0), ttm.L.TTM_OP_PEAKS, 32, tuple(s["score"].shape), device=DEV)
    elif kind == "train":
        C, u, p = _pairs(case, seed)
        net = ttm.MLP(ctx, ttm.make_desc(case["n"], 32, 14.0), p)
        net.v.fill_(1e-4)          # moments of a run under way
        net.step = 1000
        s.update(C=C, u=u, net=net, grads=torch.empty(net.n_params, device=DEV))
    elif kind == "template":
        s["tmpl"], s["quats"] = _density_box(case, seed)
        s["desc"] = ttm.make_desc(case["n"], case["L"], case["r"], dprime=case["dprime"])
    return s


# ----------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------

def run(state):
    s, case, ctx = state, state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "pass":
        p = s["engine"].run(s["vol"], top_p=case["top"])
        return dict(score=p.score, lam=p.lam, dir=p.direction, w=p.w, peaks=p.peaks, vals=p.peak_vals)
    if kind == "item":
        g, w, stats = ttm.normalize(ctx, s["desc"], s["vol"], s["spec"], case["N"])
        C = ttm.correlate(ctx, s["desc"], g, w, stats, s["spec"], case["N"], s["lo"], s["size"], dtype=s["dtype"])
        return dict(g=g, w=w, stats=stats, C=C)
    if kind == "tile":
        C = ttm.normalize_correlate(ctx, s["desc"], s["g"], s["stats"], s["spec"], case["N"], s["lo"], s["size"],
                                    s["w"], out=s["out"], ws=s["ws"])
        return dict(w=s["w"], C=C)
    if kind == "localise":
        p = s["engine"].run(s["vol"], top_p=case["grid"] ** 3)
        ref = ttm.refine(ctx, s["desc"], p.g, p.w, s["T"], s["tn"], p.peaks.contiguous(), s["starts"], r_s=3.0)
        return dict(score=p.score, w=p.w, peaks=p.peaks, vals=p.peak_vals, pos=ref["pos"], quat=ref["quat"],
                    lncc=ref["lncc"], lncc_peak=ref["lncc_peak"])
    if kind == "batch":
        be = s["engine"]
        for v, x in zip(be.volumes, s["vols"]):
            v.copy_(x)
        be.replay()
        return dict(score=be.score, lam=be.lam, dir=be.direction, peaks=be.peaks, vals=be.vals, found=be.n_found)
    if kind == "extract":
        score, lam, u = ttm.extract(ctx, s["desc"], s["C"], score=s["score"], lam=s["lam"], direction=s["dir"],
                                    starts=s["starts"], mlp=s["net"], kappa=float("-inf") if s["net"] else 0.0,
                                    fallbacks=s["fb"], ws=s["ws"])
        return dict(score=score, lam=lam, dir=u)
    if kind == "peaks":
        lo, hi = ttm.valid_bounds(s["score"].shape, case["L"])
        peaks, vals = ttm.find_peaks(ctx, s["score"], lo, hi, case["top"], 2.0 * case["r"], ws=s["ws"])
        return dict(peaks=peaks, vals=vals)
    if kind == "train":
        net = s["net"]
        loss = net.train_step(s["C"], s["u"], lr=1e-3, grads=s["grads"])
        return dict(loss=loss, grads=s["grads"], params=net.params, m=net.m, v=net.v)
    T, tn = ttm.build_tensor(ctx, s["desc"], s["tmpl"], s["quats"])
    return dict(T=T, tn=tn)


# ----------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------

def _K(n, d=3):
    return math.comb(n + d - 1, n)


def _tiles(shape, L, N):
    return math.prod(-(-(v - L + 1) // (N - L + 1)) for v in shape)


def _field_work(shape, n, d, L, N, size, tiles=None):
    """Bytes and flops of the local normalisation and the field of one volume."""
    K, V, U = _K(n, d), math.prod(shape), math.prod(v - L + 1 for v in shape)
    t = _tiles(shape, L, N) if tiles is None else tiles
    fft = 2.5 * N ** 3 * 3 * math.log2(N)
    return 4 * V + (K + 1) * L * (N // 2 + 1) * N * 8 + 4 * U + size * K * U, t * (K + 4) * fft


_PER_VOXEL = {True: 3000.0, False: 16 * 45 * 200.0}   # flops of a voxel's orientation: learned, 16 starts


def work(case):
    kind = case["kind"]
    if kind in ("pass", "item", "tile"):
        shape, n, L = _shape(case), case["n"], case["L"]
        b, f = _field_work(shape, n, 3, L, case["N"], 2 if case.get("bf16") else 4)
        V, U = math.prod(shape), math.prod(v - L + 1 for v in shape)
        if kind == "item":
            b += 4 * V + 8
        if kind == "pass":
            b += 4 * V + 20 * U - 4 * _K(n) * U
            f += U * _PER_VOXEL[False]
        return dict(bytes=b, flops=f)
    if kind == "localise":
        L, K, P = case["L"], _K(case["n"], 4), case["grid"] ** 3
        e = 2 * (L // 2 + 2) + (case["grid"] - 1) * case["spacing"] + 1
        b, f = _field_work((e,) * 3, case["n"], 4, L, case["N"], 0)
        per = K * L ** 3 * 2 + 32 * 45 * 400 + (2 * case["r"] + 5) ** 3 * 2
        return dict(bytes=b + 12 * e ** 3 + 4 * K * L ** 3, flops=f + P * 123 * per)
    if kind == "batch":
        b = f = 0
        for i, e in enumerate(int(v) for v in case["edges"].split(",")):
            L = _BATCH[i % 2][0]
            N = ttm.pick_fft((e,) * 3, L)
            x, y = _field_work((e,) * 3, case["n"], 3, L, N, 0)
            b += x + 4 * e ** 3 + 20 * (e - L + 1) ** 3
            f += y + (e - L + 1) ** 3 * _PER_VOXEL[True]
        return dict(bytes=b, flops=f)
    if kind == "extract":
        U, K = case["bz"] * case["by"] * case["bx"], _K(case["n"])
        return dict(bytes=U * (4 * K + 20), flops=U * _PER_VOXEL[case["learned"]])
    if kind == "peaks":
        return dict(bytes=4 * math.prod(v - case["L"] + 1 for v in _shape(case)) + 16 * case["top"], flops=0)
    if kind == "train":
        K, B = _K(case["n"]), case["B"]
        return dict(bytes=B * (K + 3) * 4 + 7312 * 4 * 7, flops=6 * B * (32 * 64 + 64 * 64 + 64 * 3))
    K, L = _K(case["n"], case["dprime"]), case["L"]
    inside = 4.0 / 3.0 * math.pi * (case["r"] + 1) ** 3
    return dict(bytes=4 * (K + 2) * L ** 3 + 16 * case["nq"], flops=case["nq"] * inside * (2 * K + 40))


# ----------------------------------------------------------------------------
# the outputs in 64 bits
# ----------------------------------------------------------------------------

def exact(case, seed):
    kind = case["kind"]
    if kind in ("pass", "item", "tile"):
        vol, T = _volume(case, seed)
        L = case["L"]
        g, w, stats, C = _field(vol, T, L, case["r"])
        shape = _shape(case)
        if kind == "pass":
            return dict(score=_full(_score(C, case["n"], 3), shape, L), lam=None, dir=None, w=_full(w, shape, L),
                        peaks=None, vals=None)
        if kind == "item":
            return dict(g=g, w=_full(w, shape, L), stats=stats, C=C)
        return dict(w=_full(w, shape, L), C=C)
    if kind == "localise":
        vol, T, _ = _grid_volume(case, seed)
        _, w, _, C = _field(vol, T, case["L"], case["r"])
        shape = tuple(vol.shape)
        return dict(score=_full(_score(C, case["n"], 4), shape, case["L"]), w=_full(w, shape, case["L"]), peaks=None,
                    vals=None, pos=None, quat=None, lncc=None, lncc_peak=None)
    if kind == "batch":
        out = []
        for i, v in enumerate(_batch_volumes(case, seed)):
            L, r = _BATCH[i % 2]
            C = _field(v, _template(case["n"], L, r)[1], L, r)[3]
            out.append(_full(_score(C, case["n"], 3), tuple(v.shape), L))
        return dict(score=out, lam=None, dir=None, peaks=None, vals=None, found=None)
    if kind == "extract":
        L = case["L"]
        r = float(int(0.43 * L))
        model, T, _ = _template(case["n"], L, r)
        box = (case["bz"], case["by"], case["bx"])
        C = _field(_tomogram(tuple(b + L - 1 for b in box), model, L, r, 0.1, seed), T, L, r)[3].float()
        return dict(score=_score(C, case["n"], 3), lam=None, dir=None)
    if kind == "train":
        return _train_exact(case, seed)
    if kind == "template":
        tmpl, quats = _density_box(case, seed)
        T, tn = _tensor_template(tmpl, case["L"], case["r"], quats.to(F64), case["n"], case["dprime"])
        return dict(T=T, tn=tn)
    return None


def _train_exact(case, seed):
    """One step in 64 bits, without the BF16 rounding of operands and activations."""
    C, u, p = _pairs(case, seed)
    C, u, p = C.to(F64), u.to(F64), p.to(F64).requires_grad_()
    _, mu = _exponents(case["n"], 3)
    K = C.shape[1]
    X = C * mu.sqrt()
    X = X / X.norm(dim=1, keepdim=True)
    W1, b1, W2, b2, W3, b3 = torch.split(p, [32 * 64, 64, 64 * 64, 64, 64 * 16, 16])
    h = torch.relu(torch.relu(X @ W1.view(32, 64)[:K] + b1) @ W2.view(64, 64) + b2)
    y = (h @ W3.view(64, 16) + b3)[:, :3]
    loss = (1 - ((y / y.norm(dim=1, keepdim=True)) * u).sum(1) ** 2 / (u * u).sum(1)).mean()
    loss.backward()
    g = p.grad
    m, v = 0.1 * g, 0.999 * float(np.float32(1e-4)) + 0.001 * g * g
    pad1, pad3, padb = (torch.zeros(k, dtype=torch.bool, device=DEV) for k in ((32, 64), (64, 16), (16,)))
    pad1[K:], pad3[:, 3:], padb[3:] = True, True, True       # rows and columns that stay 0
    used = torch.zeros(64, dtype=torch.bool, device=DEV)
    pad = torch.cat([pad1.flatten(), used, used.repeat(64), used, pad3.flatten(), padb])
    v = torch.where(pad, torch.zeros_like(v), v)
    t = 1001
    new = p.detach() - 1e-3 * (m / (1 - 0.9 ** t)) / (torch.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
    return dict(loss=loss.detach().view(1), grads=g, params=new, m=m, v=v)
