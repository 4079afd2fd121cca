"""Which matrices take both passes over the history in one launch, and into how many tiles they are cut: host arithmetic, on
handles that nothing launches on."""
import ctypes

import pytest

from paper_2410_16029_amd import binding as B


def _tiles(ls):
    return [B._lib.ng_debug_history_tiles(ls.st, ctypes.c_int(i)) for i in range(len(ls.shapes))]


def _set(shapes, r, **kw):
    return B.LayerSet(shapes, r, device="cpu", host_only=True, **kw)


def _expect(r, n, rows_per_lane, most):
    ldn = (n + 31) // 32 * 32
    bands = 1 if r <= 8 else 2 if r <= 16 or rows_per_lane == 2 else 4
    t = -(-r // (8 * bands)) * -(-ldn // (32 * rows_per_lane * (4 // bands)))
    return t if t <= most else 0


@pytest.mark.parametrize("dtype,hist,s,rows,most", [
    ("f32", "f32", 4, 2, 128), ("f32", "f32", 8, 2, 256), ("f32", "f32", 16, 2, 256),
    ("bf16", "f32", 3, 4, 384), ("bf16", "f32", 8, 4, 384), ("bf16", "f32", 9, 2, 512),
    ("bf16", "bf16", 4, 4, 192), ("bf16", "bf16", 5, 4, 384), ("bf16", "bf16", 16, 4, 384)])
def test_tiles_of_a_matrix(dtype, hist, s, rows, most):
    cases = [(1, 40), (8, 513), (9, 130), (16, 31), (17, 777), (64, 4096), (64, 4200), (256, 1024), (128, 1500), (256, 2752), (512, 2048), (512, 2049)]
    ls = _set([(max(r, 40), n) for r, n in cases], [r for r, _ in cases], dtype=dtype, hist_dtype=hist, s=s)
    assert _tiles(ls) == [_expect(r, n, rows, most) for r, n in cases]


@pytest.mark.parametrize("s", [0, 17, 64])
def test_none_without_history_or_beyond_its_slots(s):
    assert _tiles(_set([(64, 100), (300, 200)], 16, dtype="bf16", s=s)) == [0, 0]


def test_right_side_counts_the_projected_problem():
    # 300 x 140 on the right side: rank 24 over 300 columns
    left, right = (_set([(300, 140)], 24, dtype="bf16", s=4, sides=x) for x in (None, "right"))
    assert _tiles(left) == [_expect(24, 140, 4, 384)] and _tiles(right) == [_expect(24, 300, 4, 384)]


@pytest.mark.parametrize("tiles", [1, 24, 512])
def test_tiles_give_way_to_those_that_have_not_started(tiles):
    def leave(missing, look):
        return sum(B._lib.ng_debug_history_leaves(t, missing, look) for t in range(tiles))

    patience = 100
    for look in range(patience - 1):
        assert leave(0, look) == 0                               # all have started: nobody's place is wanted
        for missing in (1, 3, 200, tiles + 1):
            assert leave(missing, look) == min(tiles, missing << min(look, 16))
    assert leave(0, patience - 1) == leave(1, patience - 1) == tiles     # any wait ends


@pytest.mark.parametrize("count,tiles", [(400, 512), (900, 0), (1100, 512)])
def test_a_step_that_fitted_the_librarys_own_scratch_still_does(count, tiles):
    # Partial sums per tile take 64 KB of a matrix of 512 tiles at 16 slots, the plain ones 32 KB: 900 of these matrices fit
    # NG_STATIC_SCRATCH_BYTES (32 MiB) only with the plain ones, 400 with either and 1100 with neither.
    descs = B.make_descs([(512, 2016)] * count, 512)
    hp = B.ng_default_hparams()
    hp.s, hp.grad_dtype = 16, B.NG_BF16
    _, ws = B.ng_query_sizes(descs, hp)
    bufs = (B.ng_matrix_buffers * count)()
    for i in range(count):
        for b in range(B.NG_NBUF):
            bufs[i].buf[b] = 4096                    # (a host-only handle looks at the alignment alone)
    st = B.ng_init_state(descs, bufs, hp, 4096, ws, B.NG_INIT_HOST_ONLY, 0)
    assert {B._lib.ng_debug_history_tiles(st, ctypes.c_int(i)) for i in range(count)} == {tiles}
    B.ng_destroy(st)
