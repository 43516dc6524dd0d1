"""The statistics' serial steps at the edges of their staging: 256 blocks of
4096 points and 256 partial sums of as many.  A long series' windows against
the same windows of a short slice, whose statistics take one block."""
import numpy as np
import pytest
import torch

from paper_2401_13680_amd import api, synth

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
