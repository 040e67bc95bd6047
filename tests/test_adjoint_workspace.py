"""The workspace of the reverse sweep holds, beside records, state copies and cotangents, the dL/dg partials
that its line passes write (three doubles per wavefront and step of a segment) and their instance tables,
counted here from the passes' geometry (no GPU)."""
import ctypes

import pytest

from paper_1907_12834_amd import qlg as Q

TABLES = 7   # instance tables of the passes


def _windows(n, lines):
    """56-slot windows of lines laid end to end: n + 8 slots, or whole windows where those are fewer."""
    if n == 1:
        return -(-lines // 56)
    slots = min(n + 8, -(-n // 56) * 56)
    return -(-(lines * slots - 8) // 56)


def _partials(n, lines, planes, nx):
    """Wavefronts of a pass along y or z: 64 / n lines each up to three sites, else four columns of a
    window per workgroup, several columns in a run where their lines fill less than half a window."""
    if n <= 3:
        return -(-lines // (64 // n))
    groups = -(-nx // 4)
    slots = planes * min(n + 8, -(-n // 56) * 56)
    fold = 64 // slots if slots <= 32 else 1
    return 4 * -(-groups // fold) * _windows(n, planes * fold)


@pytest.mark.parametrize("ndim,nx,ny,nz", [
    (1, [100, 1, 57], None, None), (2, [300000], [1], None), (2, [150000, 3, 64], [2, 70, 3], None),
    (2, [1, 512, 130], [130, 512, 4], None), (3, [9, 64, 33], [1, 3, 17], [200, 64, 2]), (3, [1, 5], [1, 4], [1, 70]),
])
@pytest.mark.parametrize("dtype", [Q.C64, Q.C128])
def test_workspace_holds_the_passes_partials(ndim, nx, ny, nz, dtype):
    K = 3
    p, keep = Q.make_params(ndim, nx, ny, (1, -0.5, 0.5), 0.1, dtype, Q.INTERLEAVED, nz)
    sb, cb, ck, wk = (ctypes.c_size_t() for _ in range(4))
    assert Q.lib().qlg_query_sizes(ctypes.byref(p), ctypes.byref(sb), ctypes.byref(cb)) == 0
    assert Q.lib().qlg_adjoint_query(ctypes.byref(p), 7, K, ctypes.byref(ck), ctypes.byref(wk)) == 0
    copy = sb.value // 2
    lam = copy * (2 if dtype == Q.C64 else 1)
    parts = 0
    for x, y, z in zip(nx, ny or [1] * len(nx), nz or [1] * len(nx)):
        parts += _windows(x, y * z)
        parts += _partials(y, x * z, z, x) if ndim >= 2 else 0
        parts += _partials(z, x * y, y, x) if ndim == 3 else 0
    need = 2 * K * 4 * ndim * copy + 2 * copy + 2 * lam + 8 * 3 * K * parts + 4 * TABLES * (len(nx) + 1) + 8 * (4 + 3 * 256)
    assert wk.value >= need
