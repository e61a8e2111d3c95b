"""One contiguous eighth of a launch's work per XCD, by the rule: taken where no expert has more than one block (gate+up: up to 32
feature tiles; down projection with cached loads), not taken otherwise, and every row and feature tile covered exactly once either
way.  Host arithmetic only."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
from test_launch_mapping import L, _check_cover, _schedule  # noqa: E402,F401

from paper_2605_23911_amd import binding as B  # noqa: E402


def _eighths(work, n_e0):
    """Whether the workgroups with work run through ids x, x + 8, x + 16 .. tile by tile."""
    per = [[(r[2], r[4]) for r in work[x::8] if r[0]] for x in range(8)]
    return [t for p in per for t in p] == sorted(t for p in per for t in p)


@pytest.mark.parametrize("gateup,ib,wnt,N,rule", [(True, 1, True, 2048, True), (True, 1, True, 4096, True), (True, 1, True, 4160, False),
                                                   (True, 1, True, 1408, True), (False, 2, False, 7168, True), (False, 2, False, 2880, True)])
@pytest.mark.parametrize("counts", [[100] * 40, [256, 0, 1, 255] * 16, [200] * 39 + [257], [3, 0, 600, 0, 0, 40]])
def test_rule(L, gateup, ib, wnt, N, rule, counts):  # noqa: F811
    offsets, blocks, mix, heavy = _schedule(np.array(counts), 256)
    work = B.map_launch(gateup, ib, wnt, N, 256, offsets, blocks, None, heavy, cus=256, slack_blocks=5)
    _check_cover(work, offsets, counts, N, 256, (gateup, ib, wnt, N, counts))
    single = max(counts) <= 256
    if len(blocks) * ((N + 128 * ib - 1) // (128 * ib)) > 256 * 2:      # beyond a split last round
        assert _eighths(work, counts[0]) == (rule and single)
