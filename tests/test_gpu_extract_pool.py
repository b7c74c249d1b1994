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
