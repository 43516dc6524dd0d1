"""The statistics' serial steps at the edges of their staging: 256 blocks of
4096 points and 256 partial sums of as many.  A long series' windows against
the same windows of a short slice, whose statistics take one block."""
import numpy as np
import pytest
import torch

from paper_2401_13680_amd import api, synth
from paper_2401_13680_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4096, 4097, 256 * 4096 - 1, 256 * 4096, 256 * 4096 + 1, 300 * 4096 + 5])
def test_long_series_windows_equal_a_slices(n):
    m, l = 512, 480   # (the workspace holds the profiles of n / m segments)
    x = synth.regime_series(n, 5, synth.SHAPES6).x
    T = torch.from_numpy(x).cuda()
    Q = T[100:100 + m].clone()
    D = api.mpdist_profile(T, Q, l)
    D = D[0] if isinstance(D, tuple) else D
    for at in (0, n // 2, n - 2000):
        S = api.mpdist_profile(T[at:at + 2000].clone(), Q, l)
        S = S[0] if isinstance(S, tuple) else S
        e = (D[at:at + 2000 - m + 1] - S).abs().max().item()
        assert e <= 1e-4 * 2 * np.sqrt(l), (n, at, e)


def test_windows_across_the_scan_edge_equal_a_slices():
    """A slice that straddles the 256th block of 4096 points."""
    n, m, l = 300 * 4096 + 5, 512, 480
    T = torch.from_numpy(synth.regime_series(n, 5, synth.SHAPES6).x).cuda()
    Q = T[100:100 + m].clone()
    D = api.mpdist_profile(T, Q, l)
    at = 256 * 4096 - 1000
    S = api.mpdist_profile(T[at:at + 2000].clone(), Q, l)
    assert (D[at:at + 2000 - m + 1] - S).abs().max().item() <= 1e-4 * 2 * np.sqrt(l)


@pytest.mark.parametrize("n,block", [(256 * 4096 + 1, 256), (300 * 4096 + 5, 256), (300 * 4096 + 5, 300)])
def test_partials_past_the_first_256_count(n, block):
    """Points i with i / 256 = block (of ceil(n / 4096) in turn) go to that partial: a
    non-finite one is refused, and a large one raises the level below which windows
    are constant, so that every window without it is at distance sqrt(l) of a query
    whose own are not."""
    m, l, at = 512, 480, block * 256 + 7
    x = synth.regime_series(n, 5, synth.SHAPES6).x
    Q = torch.from_numpy(x[100:100 + m].copy()).cuda()
    x[at] = 1e9
    D = api.mpdist_profile(torch.from_numpy(x).cuda(), Q, l)
    far = torch.ones_like(D, dtype=torch.bool)
    far[at - m:at + 1] = False
    assert (D[far] == np.float32(np.sqrt(np.float32(l)))).all()
    for bad in (np.inf, np.nan):
        x[at] = bad
        with pytest.raises(_lib.PstError) as e:
            api.mpdist_profile(torch.from_numpy(x).cuda(), Q, l)
        assert e.value.code == _lib.PST_EINVAL
