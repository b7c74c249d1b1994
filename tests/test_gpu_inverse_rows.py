"""The field on boxes whose number of rows chooses the inverse X pass's workgroups."""
import numpy as np
import pytest

from gpu_common import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,rows,bf16", [
    (192, 1, False),      # half a block of 32: 16 rows a workgroup
    (192, 16, False),
    (192, 17, False),     # more: 32 rows a workgroup
    (192, 161, True),     # the first row of a sixth block
    (256, 208, False),    # half of a seventh block
    (256, 209, False),
    (256, 225, False),    # one row of an eighth block: 32 rows a workgroup
    (256, 225, True),     # and 16 for bfloat16
    (256, 241, True),     # 32 rows a workgroup
    (512, 33, False),     # always 16
])
def test_field_of_boxes_of_so_many_rows(N, rows, bf16):
    """correlate against direct FFT correlation in 64 bits: the FP32 transforms'
    2e-6 normwise, plus half a bfloat16 step (2^-9) per value for that store."""
    import torch
    require_gpu()
    from paper_2408_02398_amd import ttm as T
    ctx = T.Context(0)
    L, n = 9, 2
    gen = torch.Generator().manual_seed(N + rows)
    shape = (12, rows + L - 1, 40)
    vol = torch.randn(shape, generator=gen)
    Tt = torch.randn((T.n_components(n), L, L, L), generator=gen)
    d = T.make_desc(n, L, 0.45 * L)
    spec = T.template_spectra(ctx, d, Tt.cuda(), N)
    g, w, stats = T.normalize(ctx, d, vol.cuda(), spec, N)
    lo, hi = T.valid_bounds(shape, L)
    size = tuple(b - a + 1 for a, b in zip(lo, hi))
    assert size[1] == rows
    C = T.correlate(ctx, d, g, w, stats, spec, N, lo, size, dtype=torch.bfloat16 if bf16 else torch.float32)
    G = torch.fft.rfftn(g.double())
    wv = w.double()[tuple(slice(a, b + 1) for a, b in zip(lo, hi))]
    for k in range(len(Tt)):
        ref = torch.fft.irfftn(G * torch.fft.rfftn(Tt[k].cuda().double(), s=shape).conj(), s=shape)
        ref = (wv * ref[:size[0], :size[1], :size[2]]).cpu().numpy()
        err = np.linalg.norm(C[k].double().cpu().numpy() - ref) / np.linalg.norm(ref)
        assert err <= 2e-6 + (2.0 ** -9 if bf16 else 0.0)
