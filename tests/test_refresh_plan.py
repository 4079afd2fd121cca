"""Which bases of a refresh are orthonormalised in one launch (sketches of up to 32 columns and 1024 rows): host arithmetic, on
handles that nothing launches on."""
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
