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
