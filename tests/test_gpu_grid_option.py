"""PST_OPT_PROFILE_GRID limits the workgroups of the sweep's profile launch.
Every workgroup writes a scratch slot of its own, so the end of the stretch of
the workspace that a sweep writes before the untouched rest of its scratch
tells how many there were.  Tiles are striped over the workgroups, not handed
out, so that every one of them gets some."""
import ctypes

import pytest
import torch

from paper_2401_13680_amd import _lib, api, synth

pytestmark = pytest.mark.gpu

RESIDENT = {33: 1024, 150: 768, 200: 512}   # streaming workgroups of w at once


def scratch_end(m, l, n, grid):
    """Byte offset at which the longest untouched stretch of the workspace begins."""
    L = _lib.load()
    ctx = api.context(0)
    T = torch.from_numpy(synth.regime_series(n, 3, synth.SHAPES6).x).cuda()
    ms, ls = (ctypes.c_int32 * 1)(m), (ctypes.c_int32 * 1)(l)
    nb = L.pst_select_length_workspace_bytes(n, ms, 1, ls, 1)
    ws = torch.full(((nb + 255) // 256 * 64,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    options = [(_lib.PST_OPT_SWEEP_BATCHED, 1), (_lib.PST_OPT_SWEEP_GRAPH, 0), (_lib.PST_OPT_AUTOTUNE, 0),
               (_lib.PST_OPT_TUNE_GEOMETRY, 0), (_lib.PST_OPT_SWEEP_ONE_LAUNCH, 0), (_lib.PST_OPT_DYNAMIC_TILES, 0),
               (_lib.PST_OPT_PROFILE_GRID, grid)]
    best, score, recs = ctypes.c_int32(), (ctypes.c_double * 1)(), (_lib.Snippet * 1)()
    try:
        for o, v in options:
            ctx.check(L.pst_set_option(ctx.h, o, v))
        ctx.check(L.pst_select_length(ctx.h, T.data_ptr(), n, ms, 1, ls, 1, ctypes.byref(best), score, recs, None,
                                      None, ws.data_ptr(), nb))
    finally:
        L.pst_set_option(ctx.h, _lib.PST_OPT_PROFILE_GRID, 0)
        L.pst_set_option(ctx.h, _lib.PST_OPT_DYNAMIC_TILES, 1)
    touched = (ws.view(-1, 64) != 0x5A5A5A5A).any(1).nonzero().flatten()   # 256-byte blocks, ascending
    at = int((touched[1:] - touched[:-1]).argmax())
    return (int(touched[at]) + 1) * 256


@pytest.mark.parametrize("m,l,n", [(64, 32, 40_000), (299, 150, 60_000), (399, 200, 100_000)])
def test_grid_option_limits_the_workgroups(m, l, n):
    w = m - l + 1
    one, two, half, full = (scratch_end(m, l, n, g) for g in (1, 129, 257, 0))
    # slots are equally far apart; what a workgroup writes of its own varies by
    # less than a slot
    slot = (half - two) / 128
    assert abs((two - one) / 128 / slot - 1) < 0.02, (one, two, half, full)
    assert abs((full - one) / slot + 1 - RESIDENT[w]) < 0.02 * RESIDENT[w], (one, two, half, full)
