"""The two passes over the history in one launch (k_history): ragged ranks and widths around its tiles, every count of
slots on either side of what its registers hold, matrices at and just beyond the most tiles it takes, the paths
that only a crowded chip takes (forced by a waiting limit of zero), two streams at once, and graph replays."""
import ctypes

import pytest
import torch

from paper_2410_16029_amd import binding as B
from test_gpu_edge_cases import _run
from test_gpu_parity import DEV, TOL_BF16, TOL_F32, _assert_all
from test_zz_no_alloc import _twin

pytestmark = pytest.mark.gpu


def _wait(ls, ticks):
    assert B._lib.ng_debug_history_wait(ls.st, ctypes.c_uint32(ticks)) == 0


def _tiles(ls, i):
    return B._lib.ng_debug_history_tiles(ls.st, ctypes.c_int(i))


# one octet of rows, one and two bands, rows past a band; widths below, at and past a wavefront's and a tile's columns, and
# (bf16) a state in column panels
RAGGED = [(40, 5), (64, 64), (130, 75), (96, 257), (200, 333), (72, 1000), (80, 2310)]
RANKS = [5, 8, 9, 16, 17, 33, 40]


@pytest.mark.parametrize("s", [1, 2, 3, 4, 5, 8, 9, 16, 17])
@pytest.mark.parametrize("kind", ["f32", "bf16", "bf16-hist"])
def test_ragged_tiles_and_every_class_of_slots(s, kind):
    dtype = "f32" if kind == "f32" else "bf16"
    kw = {"hist_dtype": "bf16"} if kind == "bf16-hist" else {}
    # (gradients of at least the largest rank, so that no row of R is noise alone)
    ls, errs = _run(RAGGED, RANKS, s, dtype, s + 2 if s <= 5 else 4, seed=300 + s, k=40, check=[0, 2, 4, 6], **kw)
    assert [(_tiles(ls, i) > 0) == (s <= 16) for i in range(len(RAGGED))] == [True] * len(RAGGED)
    _assert_all(errs, TOL_F32 if dtype == "f32" else TOL_BF16, kind)


@pytest.mark.parametrize("s,kind,shapes,r", [
    (16, "bf16", [(512, 2048), (512, 2049), (520, 140)], [512, 512, 24]),
    (8, "bf16", [(256, 6144), (256, 6145), (300, 140)], [256, 256, 24]),
    (8, "bf16-hist", [(256, 6144), (256, 6145), (300, 140)], [256, 256, 24]),
    (4, "f32", [(64, 4096), (64, 4097), (300, 140)], [64, 64, 24])])
def test_most_tiles_and_one_column_more_in_one_set(s, kind, shapes, r):
    # the second matrix takes the separate launches, beside the others
    dtype = "f32" if kind == "f32" else "bf16"
    kw = {"hist_dtype": "bf16"} if kind == "bf16-hist" else {}
    ls, errs = _run(shapes, r, s, dtype, 3, seed=331, k=64, energy_tol=2e-2, **kw)
    assert [_tiles(ls, i) > 0 for i in range(3)] == [True, False, True]
    _assert_all(errs, TOL_F32 if dtype == "f32" else TOL_BF16, kind)


@pytest.mark.parametrize("dtype,r,s,kw", [
    ("bf16", 64, 16, {}), ("bf16", 64, 8, {}), ("bf16", 24, 4, {}), ("bf16", 64, 16, {"hist_dtype": "bf16"}),
    ("f32", 8, 4, {}), ("f32", 40, 5, {}), ("f32", 40, 16, {})])
def test_tiles_left_by_workgroups_that_gave_way(dtype, r, s, kw):
    # one of two equal sets waits for nothing: its solvers give way to the last tiles, its tiles are left to whoever comes
    # later.  Same sums in the same order: every buffer agrees bit for bit.
    t = _twin([(384, 520), (200, 2333), (520, 384), (130, 75)], r, s, dtype, seed=347, k=40, **kw)
    assert all(_tiles(t.b, i) > 0 for i in range(4))
    _wait(t.b, 0)
    for _ in range(4):
        t.step()
    t.assert_equal("gave way")


@pytest.mark.parametrize("r,s", [(8, 5), (16, 1), (8, 9), (40, 3), (40, 5), (40, 15)])
def test_what_the_new_slot_held_before_does_not_matter(r, s):
    # fp32 sets whose projection leaves row chunks: the slot is written by the launch that also reads the ring.  One of two
    # equal sets finds NaN there; slots beyond s must not bring it in with a weight of zero.
    t = _twin([(384, 520), (200, 333), (130, 75)], r, s, "f32", seed=367, k=40)
    assert all(_tiles(t.b, i) > 0 for i in range(3))
    for _ in range(s + 1):
        for i in range(3):
            slot, head = t.b.layouts[i].slot_elems, t.b.counters(i)[1]
            t.b.buffers[i][B.NG_BUF_H].view(torch.float32)[head * slot:(head + 1) * slot].fill_(float("nan"))
        t.step()
        t.assert_equal("new slot")


@pytest.mark.parametrize("dtype,r,s", [("bf16", 64, 16), ("bf16", 72, 8), ("f32", 40, 5)])
def test_nobody_gives_way_when_all_have_started(dtype, r, s):
    # Waiting limits far below what the last sums take (2 us), on a chip that has places for all: the workgroups look whether
    # the others of their matrix have started and wait on.  (When they did not look, a slow first step sent whole matrices
    # through the workgroup that solves, tile after tile: first step of the 1.1B set 32 ms.)
    t = _twin([(384, 520), (200, 2333), (520, 384), (130, 75)], r, s, dtype, seed=373, k=40)
    _wait(t.b, 200)
    ws = t.b.workspace[(-t.b.workspace.data_ptr()) % 256:]
    B._lib.ng_debug_history_lines.restype = ctypes.c_int64
    at = [B._lib.ng_debug_history_lines(t.b.st, ctypes.c_int(i)) for i in range(4)]
    assert min(at) > 0
    left = []
    for _ in range(8):
        t.step()
        torch.cuda.synchronize()
        # eight lines of 256 bytes per matrix; behind 16 weights the tiles counted in, and whether one was left
        words = [ws[a:a + 2048].view(torch.int32).view(8, 64)[:, 32:34] for a in at]
        assert [int(w[:, 0].sum()) for w in words] == [_tiles(t.b, i) for i in range(4)]
        left.append(sum(int(w[:, 1].sum()) for w in words))
    assert min(left) == 0, left                      # (a step that something else held up may have left some)
    t.assert_equal("waited on")


def test_two_streams_at_once():
    # two sets of matrices of the largest kind on two streams: their workgroups share the chip.  Against equal sets that had
    # it to themselves.
    shapes = [(512, 2048)] * 3
    made = [_twin(shapes, 512, 16, "bf16", seed=351 + i, k=64) for i in range(2)]
    grads = [[t.stream.next_set() for _ in range(3)] for t in made]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(DEV) for _ in range(2)]
    for k in range(3):
        for t, g, st in zip(made, grads, streams):
            with torch.cuda.stream(st):
                t.a.step(g[k], t.Wa, 1e-3)
    torch.cuda.synchronize()
    for t, g in zip(made, grads):
        for k in range(3):
            t.b.step(g[k], t.Wb, 1e-3)
        t.assert_equal("two streams")


def test_replays_of_a_captured_step():
    # the graph holds the table of one step: every replay is that step again, as the eager side does it with its counters
    # put back
    t = _twin([(384, 520), (200, 333), (130, 75)], 24, 8, "bf16", seed=359, k=40)
    t.step()
    G = t.stream.next_set()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        t.a.step_static(G, t.Wa, 1e-3)
    for _ in range(3):
        graph.replay()
        at = [t.b.counters(i) for i in range(3)]
        t.b.step(G, t.Wb, 1e-3)
        after = [t.b.counters(i) for i in range(3)]
        t.assert_equal("replay")
        for i in range(3):
            B.ng_set_counters(t.b.st, i, *at[i])
    for i in range(3):
        B.ng_set_counters(t.b.st, i, *after[i])
