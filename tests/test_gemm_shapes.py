"""Host arithmetic of the library: every launch shape of a projection that the dispatch
gives has a kernel, and the no-allocation step takes the calls that libcdb.h says.  CPU
only (these functions launch nothing)."""
import ctypes as C

import pytest

import cdbgen
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


class WsLayout(C.Structure):
    _fields_ = [(n, C.c_size_t) for n in ("err", "h", "h_in", "q", "x", "act", "part", "rope", "order", "kvpid", "deff",
                                          "prow", "lm", "base", "apart", "arrive", "total")]


def _need(s, n):
    """The bytes that decide whether cdb_loop_step_noalloc takes n rows, as libcdb.h states them."""
    def splits(K):
        P = 1
        while P * s.d < 8192 and K >= 2048 * P:
            P *= 2
        return P
    P = max(splits(K) for K in (s.d, s.d_ff) + ((2 * s.d,) if s.injection else ()))
    R = next(r for r in (32, 64, 128, 256) if n <= r)
    regions = [256, 4 * n * s.d, 4 * n * s.d, 4 * n * s.d, 4 * R * s.d, 2 * R * s.d_ff, 4 * n * P * s.d, 4 * n * s.head_dim,
               4 * n, 4 * n, 4 * n, 12 * n, 128 * s.vocab]
    assert abs(sum(regions) - 256 - (n * (12 * s.d + 4 * P * s.d + 4 * s.head_dim + 24) + R * (4 * s.d + 2 * s.d_ff) +
                                     128 * s.vocab)) == 0
    return sum((b + 255) // 256 * 256 for b in regions)


def test_no_allocation_limit_is_the_stated_one():
    layout = _fn("_ZN3cdb9ws_layoutERK14cdb_model_descib", WsLayout, C.c_void_p, C.c_int, C.c_bool)
    shapes = [cdbgen.TINY, cdbgen.OURO, cdbgen.HUGINN]
    for d_ff in (96, 5632, 16384, 46816, 68928):
        for H, hd in ((1, 64), (3, 96), (16, 128), (32, 128), (55, 96), (64, 128), (330, 96)):
            shapes += [cdbgen.shrink(cdbgen.OURO, d=H * hd, n_heads=H, head_dim=hd, d_ff=d_ff, injection=i) for i in (0, 1)]
    for s in shapes:
        desc = cdb.make_desc(s)
        for n in (1, 2, 19, 32, 33, 64, 65, 100, 128, 129, 223, 256):
            w = layout(C.addressof(desc), n, False)
            assert w.base == _need(s, n), (s, n)
            if w.base <= 48 << 20:
                assert w.total <= 84 << 20, (s, n)  # the static array holds every call that is accepted
    ouro = cdb.make_desc(cdbgen.OURO)
    assert layout(C.addressof(ouro), cdb.MAX_ROWS, False).base <= 48 << 20
