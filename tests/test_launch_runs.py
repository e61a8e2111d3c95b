"""Runs of consecutive positions per XCD: when the rule takes them, on both sides of each of its lines (single-block experts; gate+up by rows
per expert and feature tiles; with multi-block experts by feature tiles and rounds), and that every row and feature tile is covered exactly once
either way.  Host arithmetic only."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
from test_launch_mapping import L, _check_cover, _schedule  # noqa: E402,F401

from paper_2605_23911_amd import binding as B  # noqa: E402


def _in_runs(work, unit):
    """Whether every XCD's workgroups (ids x, x + 8, ..) walk through whole runs of `unit` positions of the tile-major launch."""
    pos = {}
    for x in range(8):
        for q, r in enumerate(work[x::8]):
            pos.setdefault((x, q // unit), []).append((int(r[2]), int(r[4])) if r[0] else None)
    order = [t for g in range(max(k[1] for k in pos) + 1) for x in range(8) for t in pos.get((x, g), []) if t is not None]
    return order == sorted(order)


@pytest.mark.parametrize("gateup,ib,wnt,N,few", [(True, 1, True, 2048, True), (True, 1, True, 4096, True), (True, 1, True, 4160, False),
                                                  (True, 1, True, 1408, True), (False, 2, False, 7168, True), (False, 2, False, 2880, True),
                                                  (False, 1, True, 2880, True), (False, 2, False, 2048, True)])
@pytest.mark.parametrize("counts", [[100] * 64, [256, 0, 1, 255] * 24, [200] * 79 + [257], [3, 0, 600, 0, 0, 40] * 20, [300] * 7])
def test_rule(L, gateup, ib, wnt, N, few, counts):  # noqa: F811
    offsets, blocks, mix, heavy = _schedule(np.array(counts), 256)
    work = B.map_launch(gateup, ib, wnt, N, 256, offsets, blocks, None, heavy, cus=256, slack_blocks=5)
    _check_cover(work, offsets, counts, N, 256, (gateup, ib, wnt, N, counts))
    tiles = (N + 128 * ib - 1) // (128 * ib)
    total = len(blocks) * tiles
    if max(counts) <= 256:                                  # tile-major positions: the runs can be read off
        if total > 512 or ib == 1:                          # beyond a split last round
            whole, unit = (total // 128 * 128, 16) if total > 256 else (len(work), len(work) // 8)
            assert _in_runs(work[:whole], unit) == few
    # multi-block experts: the order inside an expert differs, coverage is what counts (above)


@pytest.mark.parametrize("cus", [8, 24, 64, 256, 304])
@pytest.mark.parametrize("total_blocks", [1, 2, 7, 33, 64, 65])
def test_cover_at_every_remainder(L, cus, total_blocks):  # noqa: F811
    for N in (64, 640, 1408, 2048):
        counts = [17] * total_blocks
        offsets, blocks, mix, heavy = _schedule(np.array(counts), 256)
        for gateup, ib, wnt in ((True, 1, True), (False, 1, True), (False, 2, True), (False, 2, False)):
            work = B.map_launch(gateup, ib, wnt, N, 256, offsets, blocks, None, heavy, cus=cus, slack_blocks=0)
            _check_cover(work, offsets, counts, N, 256, (cus, total_blocks, N, gateup, ib, wnt))


def _taken(gateup, ib, wnt, N, counts, M=256, **kw):
    """Whether the launch is dealt in runs: one answer for all of its workgroups."""
    offsets, blocks, _, _ = _schedule(np.array(counts), M)
    work = B.map_launch(gateup, ib, wnt, N, M, offsets, blocks, runs=True, **kw)
    _check_cover(work[:, :6], offsets, counts, N, M, (gateup, ib, wnt, N, kw))
    taken = {int(r[6]) for r in work if r[0]}
    assert len(taken) == 1
    return bool(taken.pop())


@pytest.mark.parametrize("N,rows,packed,runs", [(1536, 63, True, False), (1536, 64, True, True), (1536, 4, True, False), (2048, 64, True, True),
                                                (4096, 64, True, True), (4160, 100, True, False), (1536, 63, False, False), (1536, 64, False, True),
                                                (2048, 100, False, False), (4096, 100, False, False), (1408, 100, False, True)])
def test_gate_up_needs_rows_to_share(L, N, rows, packed, runs):  # noqa: F811
    """Below 64 rows per expert (and with row-major weights at multiples of 16 feature tiles) there is too little to share, and the weight
    panels that an XCD reads at once lie in few L2 channels."""
    assert _taken(True, 1, packed, N, [rows] * 64, packed=packed) == runs
    if rows < 64:                                          # the build for two workgroups per CU holds at most 32 rows per expert
        assert not _taken(True, 1, True, N, [min(rows, 32)] * 64, M=128, half=True)


# (light blocks, blocks of two-block experts); 896 = 7 tiles, 1024 and 2048 / 2 = 8, 1408 = 11, 1792 = 14, 2560 = 20, 2880 = 23 (12 of 256), 4096 / 2 = 16
@pytest.mark.parametrize("gateup,ib,wnt,N,light,heavy,runs", [
    (False, 1, True, 896, 20, 2, True), (False, 1, True, 1024, 20, 2, True), (False, 1, True, 1792, 20, 2, True), (False, 1, True, 2048, 90, 2, False),
    (False, 1, True, 2880, 31, 2, False), (False, 1, True, 2880, 32, 2, True),     # three rounds are 768 workgroups
    (False, 2, True, 1408, 28, 4, True), (False, 2, True, 3584, 26, 4, True), (False, 2, False, 2048, 18, 2, True), (False, 2, False, 2880, 59, 4, False),
    (False, 2, False, 2880, 60, 4, True), (False, 2, False, 4096, 90, 2, False),
    (False, 2, True, 4096, 30, 2, True), (False, 2, True, 4096, 29, 2, False), (False, 1, True, 4096, 90, 2, False),   # a sixteenth of all blocks
    (True, 1, True, 1408, 91, 2, False), (True, 1, True, 1408, 92, 2, True), (True, 1, True, 1408, 60, 60, True), (True, 1, True, 1408, 61, 60, False),
    (True, 1, True, 1024, 64, 64, True), (True, 1, True, 1024, 63, 64, False), (True, 1, True, 2048, 100, 2, False), (True, 1, True, 2048, 10, 100, False),
    (True, 1, True, 2560, 24, 60, True), (True, 1, True, 2560, 25, 60, False), (True, 1, True, 2560, 80, 4, True), (True, 1, True, 2880, 20, 100, False),
    (True, 1, True, 2880, 100, 2, False)])
def test_with_multi_block_experts(L, gateup, ib, wnt, N, light, heavy, runs):  # noqa: F811
    """Two-block experts among single-block ones: both sides of every line of the rule."""
    counts = [300] * (heavy // 2) + [200] * light
    assert _taken(gateup, ib, wnt, N, counts) == runs


def _streamed(gateup, N, K, counts, ib=1):
    """Experts whose results are stored non-temporally, of those that have rows."""
    offsets, blocks, _, _ = _schedule(np.array(counts), 256)
    work = B.map_launch(gateup, ib, True, N, 256, offsets, blocks, K=K, runs=True)
    per_expert = {}
    for r in work:
        if r[0]:
            per_expert.setdefault(int(r[1]), set()).add(int(r[7]))
    assert all(len(v) == 1 for v in per_expert.values())
    return [e for e, v in sorted(per_expert.items()) if v == {1}]


def test_what_is_stored_past_the_caches(L):  # noqa: F811
    """Launches that write 2 MiB or more whose weights do not fit the Infinity Cache; single-block experts; rows of h not where an expert has
    several blocks, nor those of an expert of more than twice the mean."""
    every = list(range(8))
    for gateup in (True, False):
        assert _streamed(gateup, 4096, 4096, [32] * 8) == every                      # 2^20 values, 2^27 weights
        assert _streamed(gateup, 4096, 4096, [32] * 7 + [31]) == []                  # 2^20 - 4096 values
        assert _streamed(gateup, 4096, 2048, [200] * 8) == []                        # 2^26 weights
        assert _streamed(gateup, 4096, 2112, [200] * 8) == every
    skewed = [200] + [100] * 3 + [80, 80, 70, 70]                                    # the mean is 100
    assert _streamed(True, 4096, 4096, skewed) == every and _streamed(True, 4096, 4096, [201] + skewed[1:-1] + [69]) == every[1:]
    assert _streamed(True, 4096, 4096, [257] + [200] * 7) == [] and _streamed(False, 4096, 4096, [257] + [200] * 7) == every[1:]
    assert _streamed(False, 4096, 4096, [256, 0, 1] + [200] * 5, ib=2) == [0, 2, 3, 4, 5, 6, 7]


@pytest.mark.parametrize("ib,N,counts", [(1, 6144, [100] * 8), (2, 4096, [200] * 30), (2, 896, [17, 0, 256, 3] * 33)])
def test_row_major_down_projection_in_eighths(L, ib, N, counts):  # noqa: F811
    """One contiguous eighth of the launch per XCD where every expert is one block; runs, or none, where one has more."""
    offsets, blocks, _, _ = _schedule(np.array(counts), 256)
    work = B.map_launch(False, ib, False, N, 256, offsets, blocks, packed=False)
    _check_cover(work, offsets, counts, N, 256, (ib, N))
    assert _in_runs(work, len(work)) and not _in_runs(B.map_launch(False, ib, False, N, 256, offsets, blocks), len(work))
    counts = counts + [257]
    offsets, blocks, _, _ = _schedule(np.array(counts), 256)
    work = B.map_launch(False, ib, False, N, 256, offsets, blocks, packed=False)
    _check_cover(work, offsets, counts, N, 256, (ib, N))
    assert not _in_runs(work, len(work))


@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("gateup,ib,wnt", [(True, 1, True), (True, 1, False), (False, 1, True), (False, 1, False), (False, 2, True), (False, 2, False)])
def test_no_rows_at_all(L, gateup, ib, wnt, packed):  # noqa: F811
    """A launch sized for rows of which none came (a rank none of whose experts was chosen): no workgroup has work, nothing is divided by zero."""
    work = B.map_launch(gateup, ib, wnt, 512, 256, np.zeros(9, dtype=np.int32), np.zeros((0, 2), dtype=np.int32), packed=packed, slack_blocks=8)
    assert len(work) and not work[:, 0].any()
