"""Cost of the orientation search across the lines of the rule that sizes its pool."""
import time

import numpy as np
import pytest

from gpu_common import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dprime,n,below,above", [
    (3, 2, (62, 63, 63), (63, 64, 64)),      # 4 million runs of 16 starts
    (3, 4, (62, 63, 63), (63, 64, 64)),
    (4, 4, (62, 63, 63), (63, 64, 64)),
    (3, 6, (90, 93, 93), (92, 93, 93)),      # 350 million components
])
def test_few_more_runs_cost_little_more(dprime, n, below, above):
    """Tensors near one direction (short runs): boxes a few percent apart, on both
    sides of a line, must not differ by more than 1.35 in time."""
    import torch
    require_gpu()
    from oracle import sym
    from paper_2408_02398_amd import ttm as T
    ctx = T.Context(0)
    d = T.make_desc(n, 16, 7.0, dprime=dprime)
    rng = np.random.default_rng(n)
    st = rng.standard_normal((16, dprime))
    st = torch.from_numpy(st / np.linalg.norm(st, axis=1, keepdims=True)).float().cuda()
    v = rng.standard_normal((4096, dprime))
    few = sym.monomials(v / np.linalg.norm(v, axis=1, keepdims=True), n)
    few = torch.from_numpy(few + 0.01 * rng.standard_normal(few.shape)).float().cuda()

    def best(shape):
        V = int(np.prod(shape))
        C = few[torch.arange(V, device="cuda") % len(few)].T.reshape(-1, *shape).contiguous()
        ws = T._ws(d, 5, 0, shape, device="cuda")
        t = []
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            T.extract(ctx, d, C, starts=st, ws=ws)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t)

    assert best(above) <= 1.35 * best(below)


def _noise(n, dprime, V, seed):
    """V tensors of independent entries: the shift is large and no start is near a fixed point."""
    from oracle import sym
    return np.random.default_rng(seed).standard_normal((V, sym.n_components(n, dprime))).astype(np.float32)


def _after(C, n, dprime, starts, updates):
    """lambda after so many updates from each start in 64 bits, the largest of them, with
    the rule's shift and with the most that its bound may add (a 4096th of an interval
    of at most 4, and 1e-5)."""
    from oracle import sym
    from oracle import ttm as orc
    cn = float(sym.frobenius(C, n, dprime))
    Cu = C.astype(np.float64) / cn
    alpha = orc.unfolding_shift(Cu, n, dprime)
    return [cn * float(np.max(orc.sshopm(Cu, n, starts, al, -1.0, updates)[0])) for al in (alpha, alpha + 1e-3)]


@pytest.mark.parametrize("dprime,n,V,n_starts,updates", [
    (3, 2, 1, 1, 1),        # one run of one update
    (3, 4, 1, 1, 3),
    (3, 4, 65, 1, 2),
    (3, 6, 130, 33, 1),     # three start blocks
    (3, 6, 130, 33, 2),
    (4, 2, 40, 1, 2),
    (4, 4, 40, 17, 2),
    (4, 6, 40, 1, 3),       # pairs of wavefronts
    (4, 6, 40, 18, 4),
])
def test_runs_end_after_max_iter_updates(dprime, n, V, n_starts, updates):
    """A run that does not converge takes exactly max_iter updates and returns lambda
    after the last: FP32 sums of at most 84 terms, 1e-5 of ||C||, around the 64-bit values
    at both ends of the shift's bound."""
    import torch
    require_gpu()
    from oracle import sym
    from paper_2408_02398_amd import ttm as T
    ctx = T.Context(0)
    d = T.make_desc(n, 16, 7.0, dprime=dprime)
    C = _noise(n, dprime, V, V + n)
    rng = np.random.default_rng(n_starts)
    st = rng.standard_normal((n_starts, dprime)).astype(np.float32)
    cnt = torch.zeros(5, dtype=torch.int64, device="cuda")
    Cg = torch.from_numpy(np.ascontiguousarray(C.T).reshape(-1, 1, 1, V)).cuda()
    _, lam, u = T.extract(ctx, d, Cg, starts=torch.from_numpy(st).cuda(), max_iter=updates, tol=0.0, newton=0, counters=cnt)
    assert cnt[4].item() == V * n_starts and cnt[0].item() == V * n_starts * updates and cnt[1].item() == 0
    lam, u = lam.cpu().numpy().ravel(), u.cpu().numpy().reshape(-1, dprime).astype(np.float64)
    for v in range(V):
        ends = _after(C[v], n, dprime, st.astype(np.float64), updates)
        slack = 1e-5 * float(sym.frobenius(C[v].astype(np.float64), n, dprime))
        assert min(ends) - slack <= lam[v] <= max(ends) + slack
        assert abs(float(sym.inner_power(C[v].astype(np.float64), u[v], n)) - lam[v]) <= slack
