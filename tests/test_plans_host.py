"""Which shapes of the half-band GEMM exist, as the planners on the host ask for them."""
import ctypes as C

import pytest

from paper_2507_18181_amd import binding as B

PARTIAL, SWIGLU, QKV, RESID = range(4)


@pytest.fixture(scope="module")
def built():
    f = B.load_library()._ZN7specasr17slice_shape_builtEiii
    f.restype, f.argtypes = C.c_bool, [C.c_int] * 3
    return f


def test_only_shapes_that_a_planner_can_choose_are_built(built):
    got = {(e, hb, nc) for e in range(-1, 6) for hb in range(-1, 12) for nc in range(-1, 7) if built(e, hb, nc)}
    want = {(PARTIAL, hb, nc) for hb, nc in [(2, 1), (4, 1), (8, 1), (2, 3), (4, 3), (2, 4), (4, 4)]}
    want |= {(SWIGLU, hb, nc) for nc, top in ((1, 8), (2, 8), (3, 6)) for hb in range(1, top + 1)}
    want |= {(QKV, hb, nc) for hb in (1, 2, 3, 4) for nc in (1, 2)} | {(RESID, 1, 1), (RESID, 1, 2)}
    assert got == want


def test_where_linears_normalise_their_input():
    """Up to 1024 features, up to 256 rows or half the features, and with a gain on four elements: the linear reads it in vectors,
    any other address goes to the kernel that reads it element by element."""
    f = B.load_library()._ZN7specasr17linear_normalisesEiPKvii
    f.restype, f.argtypes = C.c_bool, [C.c_int, C.c_void_p, C.c_int, C.c_int]
    for elem in (2, 4):
        for off in range(0, 8 * elem, elem):
            for d, most in ((8, 256), (256, 256), (512, 256), (520, 260), (1024, 512), (1032, 0)):
                for rows in (1, 256, 257, 260, 261, 512, 513, 1024):
                    assert f(d, 4096 + off, elem, rows) == (rows <= most and off % (4 * elem) == 0)
