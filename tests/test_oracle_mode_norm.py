"""The oracle's mode numbers are whole, so that a mode whose |n| is the cutoff is
kept whatever N is."""
import numpy as np
import pytest

from oracle import vacuum as V


@pytest.mark.parametrize("N", [16, 25, 49, 75, 125])
def test_modes_at_the_cutoff_are_kept(N):
    nn = V.mode_norm(N)
    for n in range(1, N // 2 + 1):
        assert nn[n, 0, 0] == nn[0, n, 0] == nn[0, 0, n] == nn[-n, 0, 0] == n
        P = V.spectrum(N, 10.0, 1.0, 1.0, "field", float(n))
        assert P[n, 0, 0] > 0 and P[-n, 0, 0] > 0 and P[0, 0, n] > 0
        if n < N // 2:
            assert P[n + 1, 0, 0] == 0
