"""The size of the top-k workspace at large shapes: what the two-pass forms take
beside the norms and lists is bounded.  CPU only (no device: 256 compute units
are assumed)."""
import ctypes as C

import pytest

from paper_1810_07355_amd import _lib as L


def need(n, dim, dtype, k, nb=None):
    pitch = (dim * (4 if dtype == L.F32 else 1) + 15) // 16 * 16
    q = L.Vectors_t(0x1000, None, n, dim, dtype, pitch, L.L2SQ, 0)
    b = L.Vectors_t(0x1000 if nb is None else 0x2000, None, nb or n, dim, dtype, pitch, L.L2SQ, 0)
    return L.load().onng_topk_workspace_size(C.byref(q), C.byref(b), 0, k)


@pytest.mark.parametrize("dtype", [L.U8, L.F32])
@pytest.mark.parametrize("n", [40_000, 131_072, 200_001, 262_144, 1_000_000])
@pytest.mark.parametrize("k", [8, 100, 128, 256])
def test_general_passes(dtype, n, k):
    """Rows of more than 128 components: candidates and group minima together
    stay within 1 GiB (and a few words per row)."""
    lists = 8 * n
    assert need(n, 200, dtype, k) <= lists + (1 << 30) + 16 * n + 4096


@pytest.mark.parametrize("dtype,n,nb", [(L.F32, 10_000_000, None), (L.F32, 5_000_000, 200_000), (L.U8, 10_000_000, 400_000),
                                        (L.U8, 400_000, None)])
@pytest.mark.parametrize("k", [10, 100])
def test_wide_passes(dtype, n, nb, k):
    """Many rows of 96 components: the passes' converted queries (f32: their
    converted base as well) share memory with what only the list kernel behind
    them uses, so the size is that kernel's own (norms, lists, 256 candidate keys
    or 128 ids per row; f32: two copies of the rows), and for 32,768 query rows
    at most 2048 candidates and group minima, and 128 bytes per u8 base row."""
    b = nb or n
    lists = 4 * (n + b) + n * ((k + 7) // 8 * 8) * 8
    lists += n * 256 * 8 if dtype == L.U8 else 256 * (n + b) + n * 128 * 4
    extra = 32768 * (2048 * 12 + 8) + 4 * n + (128 * b if dtype == L.U8 else 4 * b)
    assert need(n, 96, dtype, k, nb) <= lists + extra + 8192
