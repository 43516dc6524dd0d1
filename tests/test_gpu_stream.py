"""The streaming profile kernel against the tiled one, bit for bit: both build
a cell from the same anchors by the same recurrence and select exactly, so
their profiles are the same bits.  The tiled kernel is reached through the
re-anchor period of 2^20 rows, which anchors nowhere.  Sizes at the edges of
the kernel's kinds (columns per group, keys per lane), of its strips (one
window, one short, one past) and of its lists (ties, constant stretches,
extreme order statistics, where every row of a block is listed)."""
import numpy as np
import pytest
import torch

from paper_2401_13680_amd import _lib, api, synth

pytestmark = pytest.mark.gpu

STRIP = {False: 992, True: 1984}   # windows of a strip, w <= 180 or wider


def both(call):
    ctx = api.context(0)
    ctx.check(ctx.L.pst_set_option(ctx.h, _lib.PST_OPT_ANCHOR_EVERY, 1 << 20))
    try:
        ref = call(ctx)
    finally:
        ctx.check(ctx.L.pst_set_option(ctx.h, _lib.PST_OPT_ANCHOR_EVERY, 0))
    return ref, call(ctx)


def same_set(x, m, l, k=0):
    T = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()
    (Dr, mr), (D, mx) = both(lambda c: api.profile_set(T, m, l, k, ctx=c))
    assert torch.equal(D, Dr), (m, l, k, int((D != Dr).sum()), (D != Dr).nonzero()[:3].tolist())
    assert torch.equal(mx, mr)


def series(n, seed):
    return synth.regime_series(n, seed, synth.SHAPES6, len_range=(400, 2500)).x


@pytest.mark.parametrize("w", [24, 31, 48, 58, 59, 79, 80, 116, 117, 148, 149, 180, 181, 212, 213, 264, 265, 392, 393, 513, 552])
@pytest.mark.parametrize("l", [7, 150])
def test_widths(w, l):
    m = w + l - 1
    same_set(series(4 * m + 2500, w), m, l)


@pytest.mark.parametrize("w", [48, 129, 257])
@pytest.mark.parametrize("extra", [-1, 0, 1, 13])
@pytest.mark.parametrize("strips", [1, 2, 9])
def test_ragged_strips(w, extra, strips):
    l = w - 1 if w < 200 else 64
    m = w + l - 1
    windows = strips * STRIP[w > 180] + extra
    x = series(windows + m - 1, 11)
    T = torch.from_numpy(x).cuda()
    Q = torch.from_numpy(series(m, 12)).cuda()
    ref, got = both(lambda c: api.mpdist_profile(T, Q, l, ctx=c))
    assert torch.equal(got, ref)


@pytest.mark.parametrize("m,l", [(64, 40), (128, 64), (256, 128), (400, 150), (900, 400)])
@pytest.mark.parametrize("k", ["1", "2", "w", "2w", "3w"])
def test_order_statistics(m, l, k):
    w = m - l + 1
    same_set(series(3 * m + 2100, 21), m, l, {"1": 1, "2": 2, "w": w, "2w": 2 * w, "3w": 3 * w}[k])


@pytest.mark.parametrize("m,l", [(90, 40), (200, 100), (256, 128), (500, 250), (700, 300)])
@pytest.mark.parametrize("kind", ["steps", "constant", "periodic", "noise", "walk"])
def test_ties_constants_and_noise(m, l, kind):
    n = 3 * m + 2300
    rng = np.random.default_rng(m)
    if kind == "steps":
        x = np.repeat(rng.integers(0, 3, n // 7 + 1), 7)[:n].astype(np.float64)
    elif kind == "constant":  # constant rows and columns among others
        x = series(n, 31)
        x[m // 2:2 * m] = 1.5
        x[n - m - 300:] = -2.0
    elif kind == "periodic":  # every motif repeats exactly
        x = np.tile(rng.normal(size=40), n // 40 + 1)[:n]
    elif kind == "noise":
        x = rng.normal(size=n)
    else:
        x = 40.0 * np.cumsum(rng.normal(size=n))
    same_set(x, m, l)


def test_batch_of_both_kernels_equals_each_alone():
    """A sweep and a multivariate search whose lengths need several kinds of
    kernel and the tiled one in one batch."""
    x = series(7000, 41)
    T = torch.from_numpy(x).cuda()
    ms = [50, 64, 70, 128, 200, 330, 420, 600]
    ref, got = both(lambda c: api.select_length(T, ms, 3, ctx=c))
    assert ref == got
    # in one launch every length keeps the strips it has in a launch of its own
    assert api.select_length(T, ms, 3, one_launch=True, graph=False) == got
    X = torch.from_numpy(np.stack([series(5000, 42 + j) for j in range(3)])).cuda()
    a, b = both(lambda c: api.snippets_multi(X, 256, 128, 3, ctx=c))
    assert a == b


@pytest.mark.parametrize("w", [12, 13, 17, 18, 23, 24, 29, 35, 36, 47, 79])
@pytest.mark.parametrize("k", [0, 1, 8, 9, 16, 17, 10 ** 6])
def test_narrow_widths(w, k):
    """Groups of 6 and 12 columns, k at the edges of the lists that a lane keeps."""
    l = 29
    m = w + l - 1
    k = min(k, 2 * w + 3)
    same_set(series(5 * m + 2100, w + k), m, l, k)
    x = series(2 * m + 1200, w)
    x[m:3 * m // 2] = 1.5
    x[500:] = np.tile(x[500:540], len(x) // 40 + 1)[:len(x) - 500]
    same_set(x, m, l, k)


@pytest.mark.parametrize("ms", [[30, 64], [30, 50, 100, 200], [64, 200, 330], [30, 300, 500, 900]])
def test_narrow_kinds_share_a_launch(ms):
    T = torch.from_numpy(series(4100, 43)).cuda()
    ref, got = both(lambda c: api.select_length(T, ms, 3, ctx=c))
    assert ref == got


@pytest.mark.parametrize("w", [80, 129, 180])
@pytest.mark.parametrize("k", ["1", "31", "33", "w", "2w-33", "2w-31", "2w"])
def test_long_lists(w, k):
    """Ranks on both sides of the keys that a lane keeps of a long list, from
    either end, on series whose blocks list most of their rows."""
    k = {"1": 1, "31": 31, "33": 33, "w": w, "2w-33": 2 * w - 33, "2w-31": 2 * w - 31, "2w": 2 * w}[k]
    rng = np.random.default_rng(w + k)
    m = 2 * w - 2
    n = 3 * m + 1400
    same_set(np.cumsum(rng.normal(size=n)), m, w - 1, k)
    same_set(rng.normal(size=n), m, w - 1, k)


@pytest.mark.parametrize("n,m", [(40011, 64), (60013, 256), (100000, 400)])
def test_runs_of_strips(n, m):
    """Long enough for runs of several strips and the single ones after them."""
    same_set(series(n, m), m, m // 2)


def test_runs_of_strips_in_a_batch():
    T = torch.from_numpy(series(40000, 44)).cuda()
    ref, got = both(lambda c: api.select_length(T, [64, 128], 3, ctx=c))
    assert ref == got


@pytest.mark.parametrize("w", [179, 190, 200, 230, 264])
@pytest.mark.parametrize("kind", ["period", "sine", "flat"])
@pytest.mark.parametrize("short", [False, True])
def test_equal_values_under_half_keys(w, kind, short):
    """Blocks whose open rows share one upper half: exact repeats (mostly y = 0,
    which an upper half of 0 settles) and constant stretches (y = 1/4), down to
    a last strip of one window whose groups end inside the first wave."""
    l = w // 3 if short else w - 1
    m = w + l - 1
    for windows in (1985, 2 * 1984 + 700):
        n = max(windows + m - 1, 2 * m)
        if kind == "period":
            x = np.tile(np.random.default_rng(w).normal(size=40), n // 40 + 1)[:n]
        elif kind == "sine":
            x = np.sin(np.arange(n) * 2 * np.pi / 100.0)
        else:
            x = series(n, 51)
            x[n // 4:n // 2] = 1.0
        for k in (0, 1, w // 3, w, 2 * w):
            same_set(x, m, l, k)


@pytest.mark.parametrize("w", [178, 179, 513, 514, 552, 553])
@pytest.mark.parametrize("l", [7, 150])
def test_widths_at_the_lines_of_the_dispatch(w, l):
    """Strips of 992 windows to w = 178 and from 514, of 1984 between; the tiled kernel from 553."""
    m = w + l - 1
    same_set(series(4 * m + 2500, w), m, l)


@pytest.mark.parametrize("w", [178, 514])
@pytest.mark.parametrize("extra", [-1, 0, 1, 13])
@pytest.mark.parametrize("strips", [1, 2, 9])
def test_ragged_strips_of_992(w, extra, strips):
    l = 64
    m = w + l - 1
    T = torch.from_numpy(series(strips * 992 + extra + m - 1, 11)).cuda()
    Q = torch.from_numpy(series(m, 12)).cuda()
    ref, got = both(lambda c: api.mpdist_profile(T, Q, l, ctx=c))
    assert torch.equal(got, ref)


@pytest.mark.parametrize("k", [1, 31, 33, 178, 2 * 178 - 33, 2 * 178 - 31, 2 * 178])
def test_long_lists_at_the_widest_kept(k):
    """w = 178, the widest whose long lists keep the keys of two lanes a window."""
    w = 178
    rng = np.random.default_rng(w + k)
    m = 2 * w - 2
    n = 3 * m + 1400
    same_set(np.cumsum(rng.normal(size=n)), m, w - 1, k)
    same_set(rng.normal(size=n), m, w - 1, k)
