"""The launch shapes of the projections, on the host: every shape the dispatch
gives a call has a kernel, for every width the model descriptor accepts.  CPU
only (the shape functions launch nothing)."""
import ctypes as C

import pytest

import paper_2608_09444_amd as cdb

QKV, PARTIAL, SWIGLU, STORE = range(4)
TILE_SHAPES, TILE_FIXED = 4, 5  # GemmShape.NS of the tile kernels
MAX_ROWS, MAX_PREFILL_ROWS = cdb.MAX_ROWS, cdb.MAX_PREFILL_ROWS


class GemmShape(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("N", "K", "S", "KW", "NS")]


class TileShape(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("WM", "WN", "gx", "gy", "S")]


def _fn(symbol, restype, *argtypes):
    f = getattr(cdb.lib(), symbol)  # C++ names: internal to the library
    f.restype, f.argtypes = restype, argtypes
    return f


def _projections(d, d_ff, vocab):
    """(N, K, epilogue) of a model's projections, the adapter in both of its forms."""
    return ((3 * d, d, QKV), (d, d, PARTIAL), (2 * d_ff, d, SWIGLU), (d, d_ff, PARTIAL), (d, 2 * d, PARTIAL),
            (d, 2 * d, STORE), (vocab, d, STORE))


def _check_tile(N, K, M, epi, S, two_parts, where):
    t = _fn("_ZN3cdb10tile_shapeEiiiiib", TileShape, *[C.c_int] * 5, C.c_bool)(N, K, M, epi, S, two_parts)
    if S:
        assert t.S == S, where
    # the instantiated tiles: 3 stripes, 2 for split-K partials, 4 with 3 m-tiles in one pass; q/k/v in two passes 3 x 3
    assert t.S >= 1 and (t.WN == 3 or (t.WN == 2 and epi == PARTIAL) or (t.WN, t.WM, two_parts) == (4, 3, False)), where
    assert t.WM == 3 or (t.WM == 4 and not (epi == QKV and two_parts)), where
    # the grid covers every stripe and row
    assert t.gx * t.WN * 32 >= N and t.gy * t.WM * 32 >= M, where


# long reductions onto few columns take the most splits: 16 at d_ff 16384 and d 512, 128 at 131072 and 64
@pytest.mark.parametrize("d", [64, 192, 480, 512, 768, 960, 1024, 2048, 2560, 3072, 4096, 5280, 8192])
def test_every_launch_shape_has_a_kernel(d):
    shape = _fn("_ZN3cdb10gemm_shapeEiiii", GemmShape, *[C.c_int] * 4)
    shape_mn = _fn("_ZN3cdb13gemm_shape_mnEiiii", GemmShape, *[C.c_int] * 4)
    for d_ff in (32, 96, 1024, 5632, 8192, 16384, 17920, 22016, 40928, 65536, 131072):
        for N, K, epi in _projections(d, d_ff, 49152):
            splits = set()
            for M in range(1, MAX_ROWS + 1):
                g = shape(N, K, epi, M)
                where = (d, d_ff, N, K, epi, M, g.S, g.KW, g.NS)
                splits.add((g.S, g.KW))
                assert g.KW in (4, 8) and g.S >= 1 and (epi == PARTIAL or g.S == 1), where
                if g.NS == TILE_FIXED:
                    _check_tile(N, K, M, epi, g.S, g.KW == 8, where)
                else:
                    assert g.NS in (1, 2) and M <= 128, where
            assert len(splits) == 1, (N, K, epi, splits)  # a row's sums do not follow the row count
            for M in range(33, MAX_PREFILL_ROWS + 1, 37):
                g = shape_mn(N, K, M, epi)
                assert g.NS == TILE_SHAPES
                _check_tile(N, K, M, epi, 0, False, (N, K, epi, M))
                _check_tile(N, K, M, epi, g.S, False, (N, K, epi, M))
