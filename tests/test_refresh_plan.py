"""Host arithmetic of a refresh, on handles that nothing launches on: which bases are orthonormalised in one launch (sketches of
up to 32 columns and 1024 rows), and how the clearing of the history is shared out."""
import ctypes

import pytest

from paper_2410_16029_amd import binding as B

A_AND_P, YB = 1, 2


def _one_launch(shapes, r, **kw):
    return B._lib.ng_debug_small_ortho(B.LayerSet(shapes, r, device="cpu", host_only=True, **kw).st)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shapes,r,sides,expected", [
    ([(1024, 1024)], 24, None, A_AND_P | YB),
    ([(1025, 1024)], 24, None, YB),
    ([(1024, 1025)], 24, None, A_AND_P),
    # the right side projects the transposed matrix: Ya and P have the caller's columns as rows, Yb the caller's rows
    ([(1025, 300)], 24, "right", A_AND_P),
    ([(300, 1025)], 24, "right", YB),
    ([(1024, 1024)], 24, "right", A_AND_P | YB),
    ([(5000, 300)], 24, "auto", A_AND_P),
    ([(300, 5000)], 24, "auto", A_AND_P),
    ([(300, 400), (400, 1025)], 24, [B.NG_SIDE_LEFT, B.NG_SIDE_RIGHT], YB),
    ([(300, 400), (300, 400)], [32, 33], None, 0),
])
def test_bases_in_one_launch(shapes, r, sides, expected, dtype):
    assert _one_launch(shapes, r, oversample=0, dtype=dtype, sides=sides) == expected


def _range(units, part, parts, blocks, block):
    lo, hi = ctypes.c_uint64(), ctypes.c_uint64()
    B._lib.ng_debug_clear_range(ctypes.c_uint64(units), part, parts, blocks, block, ctypes.byref(lo), ctypes.byref(hi))
    return lo.value, hi.value


@pytest.mark.parametrize("units", [16, 1008, 16 * 12345, (288 << 30) // 16])
@pytest.mark.parametrize("parts,blocks", [(1, 64), (4, 512), (7, 255), (7, 88), (60, 256), (4 * 127, 72)])
def test_every_workgroup_clears_as_much_as_any_other(units, parts, blocks):
    # one matrix or many, of one size or of several: what counts is the bytes
    at, sizes = 0, []
    for part in range(parts):
        for block in range(blocks):
            lo, hi = _range(units, part, parts, blocks, block)
            assert lo == at and hi >= lo
            at = hi
            sizes.append(hi - lo)
    # (cut at whole lines of 256 bytes, 16 units)
    assert at == units and all(x % 16 == 0 for x in sizes) and max(sizes) - min(sizes) <= 32
