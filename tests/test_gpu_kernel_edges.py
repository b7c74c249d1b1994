"""GPU parity at the edges of the kernels' tiles and of the rules that choose
them: each call against a plain 64-bit computation of the same quantity."""
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


def _normwise(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("N,n,L,shape,bf16", [
    (32, 0, 4, (32, 32, 32), False),       # one component, an odd crop (29 rows)
    (32, 2, 31, (33, 32, 35), False),      # crops of 2 rows and less over several tiles
    (64, 4, 17, (64, 50, 64), False),      # K = 15: the last component part is short
    (96, 6, 24, (96, 96, 90), False),      # odd crop of one plane per workgroup
    (96, 0, 5, (96, 95, 96), False),
    (128, 6, 31, (128, 60, 128), True),    # bfloat16 store, crop shorter than a workgroup's rows
    (128, 2, 33, (128, 128, 129), False),  # a second tile of one column
    (160, 2, 40, (160, 160, 159), False),
    (192, 2, 32, (192, 190, 192), False),  # the separate Y and X passes
])
def test_field_at_tile_edges(T, ctx, N, n, L, shape, bf16):
    """correlate against direct FFT correlation in 64 bits.  Bound: the FP32
    transforms' 2e-6 normwise (as the FFT tests), plus half a bfloat16 step
    (2^-9) per value for the bfloat16 store."""
    import torch
    gen = torch.Generator().manual_seed(N + L)
    vol = torch.randn(shape, generator=gen)
    K = T.n_components(n)
    Tt = torch.randn((K, L, L, L), generator=gen)
    d = T.make_desc(n, L, 0.45 * L)
    spec = T.template_spectra(ctx, d, Tt.cuda(), N)
    g, w, stats = T.normalize(ctx, d, vol.cuda(), spec, N)
    lo, hi = T.valid_bounds(shape, L)
    size = tuple(b - a + 1 for a, b in zip(lo, hi))
    C = T.correlate(ctx, d, g, w, stats, spec, N, lo, size, dtype=torch.bfloat16 if bf16 else torch.float32)
    G = torch.fft.rfftn(g.double())
    wv = w.double()[tuple(slice(a, b + 1) for a, b in zip(lo, hi))]
    assert float(wv.min()) > 0.0
    for k in range(K):
        ref = torch.fft.irfftn(G * torch.fft.rfftn(Tt[k].cuda().double(), s=shape).conj(), s=shape)
        ref = wv * ref[:size[0], :size[1], :size[2]]
        assert _normwise(C[k].double().cpu().numpy(), ref.cpu().numpy()) <= 2e-6 + (2.0 ** -9 if bf16 else 0.0)


def _tensor_template(tn, quats, n, d, L):
    """Alg. 1 in 64 bits: (1/nq) sum_q v_q^alpha t'(c + R_q^T (p - c)), trilinear, 0 outside the box."""
    import itertools

    from scipy.ndimage import map_coordinates
    q = quats / np.linalg.norm(quats, axis=1, keepdims=True)
    w, x, y, z = q.T
    R = np.array([[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
                  [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
                  [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]]).transpose(2, 0, 1)
    v = q if d == 4 else R[:, :, 2]
    ex = [e for e in itertools.product(range(n, -1, -1), repeat=d) if sum(e) == n]
    i = np.arange(L) - L // 2
    zz, yy, xx = np.meshgrid(i, i, i, indexing="ij")
    p = np.stack([xx, yy, zz], -1).reshape(-1, 3)
    out = np.zeros((len(ex), L ** 3))
    pad = np.pad(tn.astype(np.float64), 2)
    for k in range(len(q)):
        s = p @ R[k] + L // 2 + 2
        val = map_coordinates(pad, s[:, ::-1].T, order=1, mode="constant", cval=0.0)
        out += np.outer([np.prod(v[k] ** np.array(e)) for e in ex], val)
    return out.reshape(-1, L, L, L) / len(q)


@pytest.mark.parametrize("L,r,n,dprime,nq", [
    (2, 0.9, 2, 3, 3),       # the smallest box: every cell pair is the same one
    (7, 3.4, 0, 3, 1),       # one component, one rotation; the ball meets the box's faces
    (12, 5.9, 6, 3, 65),     # a second chunk of one rotation
    (9, 4.0, 4, 4, 300),     # 35 components: two tiles of 32, chunks on every wavefront
    (8, 3.5, 8, 4, 70),      # 165 components: a launch per 32
    (37, 17.0, 2, 3, 5),     # the largest ball that t' is kept in LDS for
    (39, 19.4, 4, 4, 67),    # t' read from memory: 35 components, two tiles at once
    (64, 31.9, 2, 3, 2),     # the largest template
])
def test_tensor_template_edges(T, ctx, L, r, n, dprime, nq):
    """build_tensor against Alg. 1 in 64 bits on its own t': 1e-5 normwise, as the parity test."""
    import torch
    rng = np.random.default_rng(L)
    tmpl = torch.from_numpy(rng.standard_normal((L, L, L)).astype(np.float32)).cuda()
    quats = rng.standard_normal((nq, 4)).astype(np.float32)
    Tt, tn = T.build_tensor(ctx, T.make_desc(n, L, r, dprime=dprime), tmpl, torch.from_numpy(quats).cuda())
    ref = _tensor_template(tn.cpu().numpy(), quats.astype(np.float64), n, dprime, L)
    got = Tt.cpu().numpy().astype(np.float64)
    if not np.linalg.norm(ref) > 0.0:
        assert np.array_equal(got, ref)
    else:
        assert _normwise(got, ref) <= 1e-5


@pytest.mark.parametrize("n,dprime,B", [(2, 3, 1), (6, 3, 15), (4, 3, 65), (4, 4, 130), (6, 3, 8193), (2, 4, 16400)])
def test_training_step_edges(T, ctx, n, dprime, B):
    """train_step's gradients and loss against the oracle's network with BF16
    operands and activations, for batches that end inside a wavefront's 16
    samples, a workgroup's 64, and past one and two blocks per workgroup.
    Bound: 1e-2 normwise, the bound of the gradient parity test (what is left
    between the two is the BF16 rounding of dY, dZ2 and dZ1 as operands, 2^-9
    each)."""
    import torch

    from oracle import mlp as omlp
    rng = np.random.default_rng(B)
    K = T.n_components(n, dprime)
    p = omlp.init_params(rng, K, d_out=dprime)
    for b in ("b1", "b2", "b3"):
        p[b] = 0.1 * rng.standard_normal(p[b].shape)
    C, t = rng.standard_normal((B, K)), rng.standard_normal((B, dprime))
    flat = omlp.pad_params(p, K, dprime).astype(np.float32)
    net = T.MLP(ctx, T.make_desc(n, 16, 7.0, dprime=dprime), torch.from_numpy(flat).cuda())
    grads = torch.empty(net.n_params, device="cuda")
    before = net.params.clone()
    loss = net.train_step(torch.from_numpy(C.astype(np.float32)).cuda(), torch.from_numpy(t.astype(np.float32)).cuda(),
                          lr=0.0, grads=grads)
    assert torch.equal(net.params, before)
    pr = {k: (omlp.bf16_round(v) if k.startswith("W") else v) for k, v in p.items()}
    y, cache = omlp.forward(pr, omlp.features(C, n, dprime), bf16=True)
    ref = omlp.pad_params(omlp.backward(pr, cache, t), K, dprime)
    assert float(loss) == pytest.approx(omlp.loss(y, t), rel=1e-3)
    assert _normwise(grads.cpu().numpy().astype(np.float64), ref) <= 1e-2


@pytest.mark.parametrize("L,r,n,n_peaks,rs", [
    (11, 4.0, 2, 3, 1.0),     # rows shorter than a block of 16, a wavefront per component tile
    (16, 6.0, 4, 140, 1.5),   # whole blocks, one wavefront for all component tiles (19 candidates)
    (35, 15.0, 2, 2, 2.0),    # rows of 2 blocks and 3 voxels; the template too large for LDS
    (18, 7.0, 6, 70, 3.0),    # 84 components, 123 candidates: the second block of tiles is partly empty
])
def test_refine_field_and_lncc_edges(T, ctx, L, r, n, n_peaks, rs):
    """refine at its tile edges: the LNCC it returns at the peaks against Eq. lncc
    at the rotation it returns, in 64 bits, and that rotation's lambda against the
    best over many rotations of the exact field (Eq. tcc).  Bounds: 1e-4 of the
    LNCC scale, the bound of the refinement parity test."""
    import torch

    import synth
    from oracle import ttm as orc
    rng = np.random.default_rng(L)
    shape = (L + 12, L + 9, L + 14)
    tmpl = synth.blob_template(np.random.default_rng(1), L, 3).volume().astype(np.float32)
    vol = rng.standard_normal(shape).astype(np.float32)
    vol[2:2 + L, 3:3 + L, 4:4 + L] += 4.0 * tmpl / tmpl.max()
    d = T.make_desc(n, L, r, dprime=4)
    Q = synth.rotation_samples(3)
    Tt, tn = T.build_tensor(ctx, d, torch.from_numpy(tmpl).cuda(), torch.from_numpy(Q).float().cuda())
    N = 64
    spec = T.template_spectra(ctx, d, Tt, N)
    g, w, stats = T.normalize(ctx, d, torch.from_numpy(vol).cuda(), spec, N)
    lo, hi = T.valid_bounds(shape, L)
    peaks = np.stack([rng.integers(a, b + 1, n_peaks) for a, b in zip(lo, hi)], 1).astype(np.int32)
    starts = torch.from_numpy(synth.start_vectors(count=16, dim=4)).cuda()
    out = T.refine(ctx, d, g, w, Tt, tn, torch.from_numpy(peaks).cuda(), starts, r_s=rs)
    g64, w64, tn64, T64 = (a.double().cpu().numpy() for a in (g, w, tn, Tt))
    c = L // 2
    qp, lp = out["quat_peak"].cpu().numpy().astype(np.float64), out["lncc_peak"].cpu().numpy()
    pos, qr, lr = out["pos"].cpu().numpy(), out["quat"].cpu().numpy().astype(np.float64), out["lncc"].cpu().numpy()
    probe = synth.random_quaternions(np.random.default_rng(2), 400)
    for i in range(0, n_peaks, max(1, n_peaks // 6)):
        for (z, y, x), q, l in ((peaks[i], qp[i], lp[i]), (pos[i], qr[i], lr[i])):
            win = g64[z - c:z - c + L, y - c:y - c + L, x - c:x - c + L]
            wv = w64[z, y, x]
            from scipy.ndimage import map_coordinates
            a, b, e, f = q / np.linalg.norm(q)
            R = np.array([[1 - 2 * (e * e + f * f), 2 * (b * e - a * f), 2 * (b * f + a * e)],
                          [2 * (b * e + a * f), 1 - 2 * (b * b + f * f), 2 * (e * f - a * b)],
                          [2 * (b * f - a * e), 2 * (e * f + a * b), 1 - 2 * (b * b + e * e)]])
            k = np.arange(L) - c
            zz, yy, xx = np.meshgrid(k, k, k, indexing="ij")
            s = np.stack([xx, yy, zz], -1).reshape(-1, 3) @ R + c + 2
            rot = map_coordinates(np.pad(tn64, 2), s[:, ::-1].T, order=1, mode="constant")
            scale = wv * np.linalg.norm(win)
            assert abs(l - wv * float(rot @ win.ravel())) <= 1e-4 * max(scale, 1.0)
            C = wv * (T64.reshape(len(T64), -1) @ win.ravel())
            lam = orc.sym.inner_power(C, q / np.linalg.norm(q), n)
            best = max(float(orc.sym.inner_power(C, p, n)) for p in probe)
            assert float(lam) >= best - 1e-4 * float(orc.sym.frobenius(C, n, 4))
    assert np.all(lr >= lp)


def _greedy(score, lo, hi, top, dist):
    """Find Peaks by its definition: the first maximum of the valid box outside
    the balls of the peaks kept so far (np.argmax takes the lowest index on ties)."""
    m = np.full(score.shape, -1.0)
    box = tuple(slice(a, b + 1) for a, b in zip(lo, hi))
    s = score[box].astype(np.float64)
    m[box] = np.where(s > 0, s, 0.0)
    zz, yy, xx = np.ogrid[:m.shape[0], :m.shape[1], :m.shape[2]]
    out = []
    while len(out) < top:
        i = int(np.argmax(m))
        z, y, x = np.unravel_index(i, m.shape)
        if m[z, y, x] < 0:
            break
        out.append((int(z), int(y), int(x)))
        m[(zz - z) ** 2 + (yy - y) ** 2 + (xx - x) ** 2 < dist * dist] = -1.0
        m[z, y, x] = -1.0
    return out


@pytest.mark.parametrize("kind,shape,top,dist", [
    ("noise", (20, 30, 70), 40, 6.0),        # fewer voxels than candidates are wanted: every voxel settles
    ("noise", (40, 61, 130), 2000, 3.0),     # thousands of peaks, long chains of waiting candidates
    ("constant", (30, 40, 50), 2048, 4.0),   # ties only: the visiting order is the index order
    ("constant", (110, 104, 103), 12, 30.0), # more tied candidates than settle in parallel: the sorted walk
    ("ramp", (16, 20, 400), 60, 7.0),        # one chain: each candidate waits for its neighbour
    ("flat", (33, 40, 64), 50, 5.0),         # peaks on an exact zero background, fewer than asked for above it
    ("dense", (24, 25, 24), 2048, 0.0),      # distance 0: every voxel is a peak (the most grid cells)
    ("blobs", (150, 200, 230), 300, 9.0),    # the threshold's two levels (every voxel counted: a sample is taken from 2^23 on)
])
def test_find_peaks_candidates(T, ctx, kind, shape, top, dist):
    """find_peaks against the rule's definition, bit for bit."""
    import torch
    rng = np.random.default_rng(sum(shape))
    if kind == "constant":
        s = np.full(shape, 0.25, dtype=np.float32)
    elif kind == "ramp":
        s = np.broadcast_to(np.linspace(1.0, 2.0, shape[2], dtype=np.float32), shape).copy()
    elif kind == "flat":
        s = np.zeros(shape, dtype=np.float32)
        s.ravel()[rng.integers(0, s.size, 30)] = rng.uniform(0.1, 1.0, 30).astype(np.float32)
        s[5, 6, 7], s[0, 0, 0] = np.nan, -1.0
    else:
        s = rng.uniform(0.1, 0.2, shape).astype(np.float32)
        if kind == "blobs":
            k = np.exp(-(np.arange(-5, 6) ** 2) / 8.0)
            b = (k[:, None, None] * k[None, :, None] * k[None, None, :]).astype(np.float32)
            for _ in range(250):
                z, y, x = (int(rng.integers(5, d - 6)) for d in shape)
                s[z - 5:z + 6, y - 5:y + 6, x - 5:x + 6] += rng.uniform(0.2, 0.9) * b
    lo, hi = (2, 1, 3), tuple(d - 3 for d in shape)
    peaks, vals = T.find_peaks(ctx, torch.from_numpy(s).cuda(), lo, hi, top, dist)
    ref = _greedy(s, lo, hi, top, dist)
    assert peaks.cpu().numpy().tolist() == [list(p) for p in ref]
    assert np.array_equal(vals.cpu().numpy(), np.array([max(s[p], 0.0) if s[p] == s[p] else 0.0 for p in ref], np.float32))


@pytest.mark.parametrize("dprime,n,shape,cuts,n_starts,max_iter", [
    (3, 2, (1, 1, 1), (), 1, 500),                  # one run
    (3, 4, (1, 1, 65), (), 17, 500),                # a second start block of one start
    (3, 4, (27, 30, 30), (1, 9), 16, 500),          # 388 800 runs against 14 400 and more
    (3, 6, (9, 31, 64), (4,), 33, 3),               # runs that end at max_iter, three start blocks
    (3, 6, (40, 40, 40), (20,), 16, 500),           # 1 024 000 runs against 512 000
    (4, 2, (3, 5, 7), (1,), 5, 500),
    (4, 4, (24, 30, 32), (10,), 16, 500),           # 368 640 runs against 153 600 and 215 040
    (4, 6, (5, 9, 17), (2, 3), 18, 4),              # pairs of wavefronts, a block of two starts
])
def test_extract_runs_edges(T, ctx, dprime, n, shape, cuts, n_starts, max_iter):
    """A run's answer depends on its voxel and start alone: the box extracted
    whole equals the box in slabs, bit for bit, and takes as many updates.
    Sampled voxels (a planted direction with noise, one zero tensor) against the
    64-bit iteration from that direction: FP32 sums of at most 56 terms, 1e-5
    of lambda, and 0.05 degrees."""
    import torch

    from oracle import sym
    from oracle import ttm as orc
    d = T.make_desc(n, 16, 7.0, dprime=dprime)
    rng = np.random.default_rng(5)
    V = int(np.prod(shape))
    vs = rng.standard_normal((V, dprime))
    vs /= np.linalg.norm(vs, axis=1, keepdims=True)
    C = rng.uniform(0.5, 2.0, V)[:, None] * (sym.monomials(vs, n) + 0.004 * rng.standard_normal((V, sym.n_components(n, dprime))))
    if V > 1:
        C[V // 2] = 0.0
    Cg = torch.from_numpy(np.ascontiguousarray(C.T).reshape(-1, *shape)).float().cuda()
    st = rng.standard_normal((n_starts, dprime))
    st = torch.from_numpy(st / np.linalg.norm(st, axis=1, keepdims=True)).float().cuda()

    def run(Cf):
        cnt = torch.zeros(5, dtype=torch.int64, device="cuda")
        out = T.extract(ctx, d, Cf.contiguous(), starts=st, max_iter=max_iter, counters=cnt)
        return [x.cpu().numpy() for x in out], cnt.cpu().numpy()

    (score, lam, u), cnt = run(Cg)
    edges = [0, *cuts, shape[0]]
    parts = [run(Cg[:, a:b]) for a, b in zip(edges, edges[1:])]
    for i, whole in enumerate((score, lam, u)):
        assert np.array_equal(whole, np.concatenate([p[0][i] for p in parts]))
    assert np.array_equal(cnt, sum(p[1] for p in parts))
    assert cnt[4] == (V - (V > 1)) * n_starts and cnt[0] <= cnt[4] * max_iter
    if max_iter < 500:
        return
    lam, u = lam.ravel(), u.reshape(-1, dprime)
    if V > 1:
        assert lam[V // 2] == 0 and not u[V // 2].any()
    C64 = Cg.cpu().numpy().reshape(len(C[0]), V).T.astype(np.float64)
    for v in rng.choice(V, min(V, 24), replace=False):
        if not C64[v].any():
            continue
        ref, ur, *_ = orc.sshopm(C64[v], n, vs[v], 0.0, 1e-15, 500)
        if n_starts > 1:
            assert lam[v] >= ref * (1 - 1e-5)
        if lam[v] <= ref * (1 + 1e-5) and n_starts > 1:
            assert abs(ur @ u[v]) >= np.cos(np.radians(0.05)) * np.linalg.norm(ur)


@pytest.mark.parametrize("kind,shape,lo,hi,top,dist", [
    ("ties", (17, 25, 9), (0, 0, 0), (16, 24, 8), 512, 0.0),          # the most peaks of the keys in LDS
    ("ties", (17, 25, 9), (0, 0, 0), (16, 24, 8), 513, 0.0),          # one more
    ("ties", (40, 33, 70), (3, 0, 5), (39, 31, 60), 90, 7.3),         # many equal scores, ragged blocks
    ("flat", (24, 24, 24), (0, 0, 0), (23, 23, 23), 40, 9.0),         # one score: linear order, blocks emptied
    ("negative", (9, 10, 11), (1, 1, 1), (8, 8, 8), 30, 2.5),         # scores of 0 and less rank alike
    ("ties", (1, 1, 40), (0, 0, 0), (0, 0, 39), 9, 1.5),
    ("blobs", (208, 216, 216), (0, 0, 0), (207, 215, 215), 25, 28.0),  # 18 954 blocks: keys in global memory
    ("blobs", (200, 208, 208), (1, 1, 1), (199, 206, 207), 25, 28.0),  # 16 900: in LDS
])
def test_find_peaks_batch_edges(T, ctx, kind, shape, lo, hi, top, dist):
    """Find Peaks of a batch (the map, and a second of one voxel) is the greedy
    rule's result exactly."""
    import torch
    rng = np.random.default_rng(3)
    s = rng.uniform(0, 1, shape).astype(np.float32)
    if kind == "ties":
        s = np.round(s, 2)
    elif kind == "flat":
        s[:] = 0.5
    elif kind == "negative":
        s = np.round(s - 0.6, 1)
    elif kind == "blobs":
        from scipy.ndimage import gaussian_filter
        s = gaussian_filter(s, 3.0).astype(np.float32)
    one = np.full((1, 1, 1), 2.0, np.float32)

    def entry(a, lo, hi, top, dist):
        return dict(score=torch.from_numpy(a).cuda(), lo=lo, hi=hi, top_p=top, min_dist=dist,
                    peaks=torch.zeros((top, 3), dtype=torch.int32, device="cuda"),
                    vals=torch.zeros(top, dtype=torch.float32, device="cuda"),
                    n_found=torch.zeros(1, dtype=torch.int32, device="cuda"))
    es = [entry(s, lo, hi, top, dist), entry(one, (0, 0, 0), (0, 0, 0), 3, 1.0)]
    pb = T.PeakBatch(ctx, es)
    for _ in range(2):
        pb.run()
        torch.cuda.synchronize()
        for e, a in zip(es, (s, one)):
            ref = _greedy(np.maximum(a, 0.0), e["lo"], e["hi"], e["top_p"], e["min_dist"])
            n = int(e["n_found"].item())
            assert n == len(ref)
            got = e["peaks"][:n].cpu().numpy()
            assert np.array_equal(got, np.asarray(ref).reshape(-1, 3))
            assert np.array_equal(e["vals"][:n].cpu().numpy(), a[tuple(got.T)])


@pytest.mark.parametrize("N,L,shape", [
    (160, 24, (33, 160, 45)),     # sums stored, then combined
    (192, 24, (30, 192, 40)),     # 169 rows: the last workgroup of 8 holds one
    (192, 32, (192, 38, 33)),     # 7 rows and 2 columns
    (256, 17, (20, 40, 256)),     # 24 rows, 240 columns
    (256, 24, (25, 300, 26)),     # two tiles, the second of 44 rows
])
def test_local_deviation_rows(T, ctx, N, L, shape):
    """w of ttm_normalize against 64-bit sums over the mask of the filtered volume.
    FP32 transforms of the sums: 2e-6 of the largest local sums, noise of
    variance near its second moment, so 2e-5 of w."""
    import torch

    from scipy.signal import fftconvolve
    r = 0.43 * L
    d = T.make_desc(2, L, r)
    rng = np.random.default_rng(8)
    vol = torch.from_numpy(rng.standard_normal(shape).astype(np.float32)).cuda()
    K = T.n_components(2)
    spec = T.template_spectra(ctx, d, torch.zeros((K, L ** 3), device="cuda"), N)
    g, w, _ = T.normalize(ctx, d, vol, spec, N)
    g, w = g.cpu().numpy().astype(np.float64), w.cpu().numpy()
    i = np.arange(L) - L // 2
    m = (i[:, None, None] ** 2 + i[:, None] ** 2 + i ** 2 <= np.float32(r) ** 2).astype(np.float64)
    f = m[::-1, ::-1, ::-1]
    s1, s2 = fftconvolve(g, f, "valid"), fftconvolve(g * g, f, "valid")
    ref = 1.0 / np.sqrt(s2 - s1 * s1 / m.sum())
    c = L // 2
    box = w[c:c + ref.shape[0], c:c + ref.shape[1], c:c + ref.shape[2]]
    assert np.max(np.abs(box - ref) / ref) < 2e-5
