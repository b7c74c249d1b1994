"""The tensor template on both sides of the rule that puts t' into LDS, against Alg. 1 in
64 bits on its own t'."""
import numpy as np
import pytest

from gpu_common import require_gpu
from test_gpu_kernel_edges import _normwise, _tensor_template

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,r,n,dprime,nq", [
    (2, 0.9, 2, 3, 17),      # the smallest box, t' in LDS
    (7, 3.4, 0, 3, 17),      # the ball meets the box's faces
    (9, 4.0, 4, 4, 16),      # the most rotations that read t' from memory: 35 components
    (9, 4.0, 4, 4, 17),      # one more: two launches of 32 components
    (37, 17.0, 2, 3, 17),    # the largest ball in LDS
])
def test_template_of_so_many_rotations(L, r, n, dprime, nq):
    """1e-5 normwise, as the parity test; exactly 0 where nothing reaches."""
    import torch
    require_gpu()
    from paper_2408_02398_amd import ttm as T
    rng = np.random.default_rng(L + nq)
    tmpl = torch.from_numpy(rng.standard_normal((L, L, L)).astype(np.float32)).cuda()
    quats = rng.standard_normal((nq, 4)).astype(np.float32)
    torch.full((T.n_components(n, dprime) * L ** 3,), float("nan"), device="cuda")   # memory that is taken next holds no zeros
    Tt, tn = T.build_tensor(T.Context(0), T.make_desc(n, L, r, dprime=dprime), tmpl, torch.from_numpy(quats).cuda())
    ref = _tensor_template(tn.cpu().numpy(), quats.astype(np.float64), n, dprime, L)
    got = Tt.cpu().numpy().astype(np.float64)
    if not np.linalg.norm(ref) > 0.0:
        assert np.array_equal(got, ref)
    else:
        assert _normwise(got, ref) <= 1e-5
    i = np.arange(L) - L // 2
    far = (i[:, None, None] ** 2 + i[:, None] ** 2 + i ** 2) > (r + 2.0) ** 2
    assert not got[:, far].any()
