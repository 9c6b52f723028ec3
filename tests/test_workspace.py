"""Device memory of operators, by the library's own query (host code only).

A 3D operator has one layout, so its memory is nobody's choice: in FP32 and
FP64 it is not above what complete lists took (286 and 314 bytes a point),
and in 16 bits it has the merged weights (36 bytes), the listed edges' bits
and the diagonal's FP64 part on top of 202."""
import ctypes
import os

import pytest

from paper_1301_3925_amd import capi


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(capi.LIB_PATH):
        from paper_1301_3925_amd import build
        build.build()
    return capi.load()


def _per_point(lib, dims, storage, flags):
    g = capi.Grid()
    g.dim, g.boundary = len(dims), capi.NEUMANN
    n = 1
    for k, d in enumerate(dims):
        g.n[k] = d
        n *= d
    nb = ctypes.c_size_t()
    assert lib.adlbr_operator_workspace(ctypes.byref(g), storage, flags, ctypes.byref(nb)) == 0
    return nb.value / n


@pytest.mark.parametrize("storage,lists", [(capi.F64, 314.1), (capi.F32, 286.1),
                                           (capi.BF16, 248.1), (capi.F16, 248.1)])
@pytest.mark.parametrize("dims", [(160, 160, 160), (131, 97, 113)])
def test_3d_memory(lib, dims, storage, lists):
    assert _per_point(lib, dims, storage, 0) <= lists
    assert _per_point(lib, dims, storage, capi.OP_WIDE) <= lists + 12.1
    if storage != capi.F64:
        assert _per_point(lib, dims, storage, capi.OP_TILED) <= lists


def test_2d_memory(lib):
    """Merged pairs cost the edge weights and records, less the ranks that
    share the records' place (not with ADLBR_OP_RECORDS)."""
    plain = _per_point(lib, (2048, 2048), capi.F32, 0)
    assert plain == pytest.approx(56.3, abs=0.1)
    assert _per_point(lib, (2048, 2048), capi.F32, capi.OP_MERGED) == pytest.approx(plain + 75)
    assert _per_point(lib, (2048, 2048), capi.F32, capi.OP_RECORDS) == pytest.approx(plain + 81)
