"""The multi-source network's choices on graphs other than R-MAT: recorded levels
(frontier, its entries, vertices listed so far, pairs not reached) with the device
times of both directions.  Choosing by the network costs at most a tenth more than
the better direction of each level: two timings of one level differ by up to 5%, so
that a choice between directions that close can go either way, in both timings."""
import json

import numpy as np
import pytest

from oracle import mlp_ref
from paper_1906_03113_amd import selector as S

# name: n, entries, sources, [(level, frontier, entries, listed, unsettled, push us, pull us)]
LEVELS = {
    "random, 1,000,000 x 30, 2 sources": (1000000, 29999512, 2, [
        (0, 2, 68, 2, 1999998, 15.0, 188.5),
        (1, 68, 2119, 70, 1999930, 15.9, 197.5),
        (2, 2049, 63762, 2119, 1997879, 46.9, 220.0),
        (3, 59798, 1851218, 61917, 1937118, 313.1, 358.2),
        (4, 818270, 24835761, 880187, 780736, 999.1, 183.5),
        (5, 623888, 18271732, 1504075, 0, 241.6, 46.0),
    ]),
    "attached, 300,000 x 3, 16 sources": (300000, 1799728, 16, [
        (0, 16, 65, 16, 4799984, 15.8, 73.4),
        (1, 64, 2633, 80, 4799919, 81.2, 79.5),
        (2, 2545, 47241, 2625, 4797182, 169.9, 97.6),
        (3, 40168, 425029, 42793, 4742559, 316.1, 104.6),
        (4, 212495, 1445092, 255288, 4112985, 825.7, 76.3),
        (5, 299299, 1786569, 554587, 1817084, 724.5, 63.8),
        (6, 283513, 1512565, 838100, 146876, 215.9, 45.0),
        (7, 85888, 331166, 923988, 140, 28.1, 22.9),
        (8, 139, 431, 924127, 0, 14.6, 22.2),
    ]),
    "mesh with diagonals, 500 x 500, 16 sources": (250000, 1994004, 16, [
        (0, 16, 128, 16, 3999984, 14.8, 29.6),
        (41, 4456, 35612, 97875, 3901645, 31.2, 40.7),
        (82, 8169, 65304, 362759, 3634360, 30.8, 41.0),
        (123, 11142, 89076, 768928, 3221728, 31.6, 42.1),
        (164, 12952, 103538, 1269831, 2712675, 32.5, 42.5),
        (205, 13038, 104214, 1816424, 2157044, 32.9, 42.0),
        (246, 12247, 97880, 2335120, 1631258, 32.8, 42.6),
        (287, 10800, 86310, 2831047, 1130120, 31.9, 42.2),
        (328, 7917, 63258, 3220094, 737757, 31.1, 40.9),
        (369, 5854, 46772, 3513573, 442345, 31.5, 39.8),
        (410, 3985, 31832, 3714948, 240000, 30.6, 39.1),
        (451, 2992, 23900, 3861933, 92500, 30.9, 42.3),
    ]),
}


@pytest.mark.parametrize("name", list(LEVELS))
def test_choices_cost_little(name):
    n, nnz, q, rows = LEVELS[name]
    level, frontier, entries, listed, unsettled, push, pull = (np.array(c) for c in zip(*rows))
    X = S.ms_features(frontier, entries, listed, unsettled, [q] * len(rows), level, n, nnz)
    w = np.asarray(json.load(open(S.MS_WEIGHTS))["weights"], np.float32)
    T = np.log(np.stack([push, pull, np.ones(len(rows))], axis=-1))
    T = np.exp(S.ms_with_round_trips(X, T))[:, :2]
    choice = np.argmin(mlp_ref.forward(w, X)[0][:, :2], axis=1)
    spent = T[np.arange(len(rows)), choice].sum()
    assert spent <= 1.1 * T.min(axis=1).sum(), f"{spent:.0f} us, {T.min(axis=1).sum():.0f} at best"
