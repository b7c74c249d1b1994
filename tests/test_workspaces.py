"""Workspace sizes of the C ABI (host only)."""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2408_02398_amd", "libttm.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libttm.so not built")


def _size(desc, op, n, nz, ny=1, nx=1):
    from paper_2408_02398_amd import _lib as L
    return L.load().ttm_workspace_size(ctypes.byref(desc), op, n, nz, ny, nx)


@pytest.mark.parametrize("degree,dprime", [(6, 3), (4, 4)])
def test_training_workspace_serves_smaller_batches(degree, dprime):
    """A workspace taken for a batch of B samples serves every smaller one."""
    from paper_2408_02398_amd import _lib as L
    from paper_2408_02398_amd import ttm
    d = ttm.make_desc(degree, 16, 7.0, dprime=dprime)
    sizes = [_size(d, L.TTM_OP_MLP_TRAIN, 0, B) for B in
             (1, 64, 65, 4096, 8191, 8192, 8193, 12000, 12288, 16384, 16385, 24577, 100000, 1 << 20)]
    assert sizes == sorted(sizes)
    assert sizes[0] > 0


@pytest.mark.parametrize("N,L", [(160, 24), (192, 24), (256, 40), (512, 40)])
def test_normalisation_workspace_holds_what_is_stored(N, L):
    """Spectra, the prefilter's partial sums, and the two local sums up to edge 160 only:
    from 192 on the inverse pass forms w from them and stores neither."""
    from paper_2408_02398_amd import _lib as lib
    from paper_2408_02398_amd import ttm
    d = ttm.make_desc(6, L, 0.4 * L)
    spec = (N * (N // 2 + 1) * N * 8 + 255) // 256 * 256
    sums = 2 * (((N - L + 1) ** 3 * 4 + 255) // 256 * 256) if N <= 160 else 0
    assert _size(d, lib.TTM_OP_NORM_CORR, N, 0, 0, 0) == (2 + 28) * spec + sums
    assert _size(d, lib.TTM_OP_NORMALIZE, N, N, N, N) == 4 * spec + sums + _size(d, lib.TTM_OP_PREFILTER, 0, N, N, N)
