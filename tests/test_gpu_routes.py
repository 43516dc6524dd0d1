"""A profile set on both sides of the line between the two profile kernels, in
launches that fill the chip: the same bits as the tiled kernel alone (reached
through the re-anchor period of 2^20 rows, which anchors nowhere), also where
jobs of both kernels share a batch."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2401_13680_amd import _lib, api, synth

pytestmark = pytest.mark.gpu


def both(call):
    ctx = api.context(0)
    ctx.check(ctx.L.pst_set_option(ctx.h, _lib.PST_OPT_ANCHOR_EVERY, 1 << 20))
    try:
        ref = call(ctx)
    finally:
        ctx.check(ctx.L.pst_set_option(ctx.h, _lib.PST_OPT_ANCHOR_EVERY, 0))
    return ref, call(ctx)


def streams(w, k, Nm, nq):
    return bool(_lib.load().pst_host_streams(ctypes.c_int32(w), ctypes.c_int32(k), ctypes.c_int64(Nm),
                                             ctypes.c_int64(nq)))


@pytest.mark.parametrize("w,line", [(17, 16), (33, 11), (47, 16), (65, 26), (129, 77), (265, 132)])
def test_both_sides_of_the_line(w, line):
    m, l = 2 * w - 1, w
    n = 42_000 if w > 178 else 31_000
    T = torch.from_numpy(synth.regime_series(n, w, synth.SHAPES6, len_range=(400, 2500)).x).cuda()
    for k in (line, line + 1, 2 * w):
        assert streams(w, k, n - m + 1, n // m) == (k == line or (k == 2 * w and w not in (33, 265))), (w, k)
        (Dr, mr), (D, mx) = both(lambda c: api.profile_set(T, m, l, k, ctx=c))
        assert torch.equal(D, Dr) and torch.equal(mx, mr), (w, k, int((D != Dr).sum()))


def test_jobs_of_both_kernels_in_a_batch():
    """Two lengths of one geometry, one on each side of the line: w = 33 at its
    default rank of 13 (l = 3/4 m) and w = 64 at 13."""
    ms, ls = [128, 127], [96, 64]
    n = 60_000
    assert not streams(33, 13, n - 127, n // 128) and streams(64, 13, n - 126, n // 127)
    assert api.geometry(33) == api.geometry(64)
    T = torch.from_numpy(synth.regime_series(n, 7, synth.SHAPES6, len_range=(400, 2500)).x).cuda()
    ref, got = both(lambda c: api.select_length(T, ms, 3, l_list=ls, ctx=c))
    assert got == ref
    assert api.select_length(T, ms, 3, l_list=ls, batched=False) == got


def test_resident_workgroups_are_the_runtimes():
    """What the launches plan for against the runtime's count, at every width."""
    L = _lib.load()
    torch.cuda.init()
    plan = {w: L.pst_host_stream_resident(ctypes.c_int32(w)) for w in range(12, 553)}
    got = {w: L.pst_device_stream_resident(ctypes.c_int32(w)) for w in plan}
    assert got == plan, {w: (plan[w], got[w]) for w in plan if got[w] != plan[w]}


def scores(T, ws, ctx=None, **kw):
    """Scores of the lengths whose windows hold w = l + 1 subsequences."""
    ms, ls = [2 * w - 2 for w in ws], [w - 1 for w in ws]
    return api.select_length(T, ms, 3, l_list=ls, ctx=ctx, **kw)["scores"]


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("ws", [[9, 51], [9, 51, 201, 301, 531, 601], [531, 601], [9, 11]])
def test_widths_of_both_kernels_in_one_launch(ws, graph):
    """w = 9 and 601 are the tiled kernel's, the others stream; past w = 513 the
    strips and tiles of every width are those of a launch of its own, so all scores
    are the tiled kernel's, bit for bit.  Twice, with other work between."""
    T = torch.from_numpy(synth.regime_series(6000, 45, synth.SHAPES6, len_range=(400, 2500)).x).cuda()
    ref, got = both(lambda c: scores(T, ws, ctx=c, one_launch=True, graph=graph))
    assert got == ref
    alone = scores(T, ws, batched=False)
    assert scores(T, ws, one_launch=True, graph=graph) == got
    split = scores(T, ws, graph=graph)
    assert split == alone and scores(T, ws, graph=graph) == alone


@pytest.mark.parametrize("graph", [False, True])
def test_widths_of_both_kernels_beside_wide_strips(graph):
    """Beside w = 301 (strips of 1984) the streaming widths up to 178 keep their own
    strips and so their own bits; w = 9 runs in the tiles of w = 301."""
    ws = [9, 51, 201, 301]
    T = torch.from_numpy(synth.regime_series(6000, 46, synth.SHAPES6, len_range=(400, 2500)).x).cuda()
    got = scores(T, ws, one_launch=True, graph=graph)
    alone = scores(T, ws, batched=False)
    assert got[1:] == alone[1:]
    assert abs(got[0] - alone[0]) <= 1e-4 * max(1.0, abs(alone[0]))
    assert scores(T, ws, one_launch=True, graph=graph) == got


def test_server_batches_of_both_kernels():
    """Requests of one shape that need both kernels, submitted together."""
    specs = [(16, 8), (100, 50), (40, 20), (1060, 530), (1200, 600), (16, 8), (128, 96)]
    xs = [torch.from_numpy(synth.regime_series(6000 + 500 * i, 47 + i, synth.SHAPES6, len_range=(400, 2500)).x).cuda()
          for i in range(len(specs))]
    srv = api.Server(0)
    tickets = [srv.submit(x, m, l, 3) for x, (m, l) in zip(xs, specs)]
    srv.drain()
    got = [srv.poll(t) for t in tickets]
    srv.close()
    for g, x, (m, l) in zip(got, xs, specs):
        assert g["status"] == 0 and g["records"] == api.snippets(x, m, l, 3)["records"], (m, l)
