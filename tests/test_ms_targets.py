"""The multi-source network's targets: device times, with a pull's round trip to the
host added from the level where pushes go in groups."""
import numpy as np

from paper_1906_03113_amd import selector as S


def test_round_trips_join_late_pulls_only():
    levels = [0, 1, S.MS_GROUP_FROM - 1, S.MS_GROUP_FROM, 700]
    n = len(levels)
    X = S.ms_features([50] * n, [300] * n, [400] * n, [9000] * n, [16] * n, levels, 1000, 8000)
    T = np.log(np.tile([20.0, 15.0, 1.0], (n, 1)))
    got = np.exp(S.ms_with_round_trips(X, T))
    want = np.tile([20.0, 15.0, 1.0], (n, 1))
    want[3:, 1] += S.MS_ROUND_TRIP
    assert np.allclose(got, want, rtol=1e-12)
    assert np.allclose(np.exp(T[:, 1]), 15.0)          # the caller's targets stay
