"""Staleness rows of every kind of end, through the step alone, the selections
and the scores (both kernel families: up to twelve views, and more): rows
shorter than a lane's 8 or 32 tokens, rows that end at or around a dword, a
lane's tokens, a pair word or an item of 64 words, at several byte offsets;
bit-exact against the oracle, and nothing written around the rows.  Scores of
few and many sets with more than twelve views: the sets' views and the step's
anchors apart, items below and above the pass's blocks."""
import numpy as np
import pytest
import torch

import oracle

from test_gpu_coverage_layouts import device_stale, random_case

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def gc():
    import paper_2608_13255_amd as gc
    return gc


@pytest.mark.parametrize("N", [3, 13])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17, 24, 29, 31, 32, 33, 34, 35, 36, 39, 40, 41, 47, 48,
                               49, 61, 62, 63, 64, 65, 80, 2016, 2031, 2032, 2047, 2048, 2049, 2064, 3600])
def test_row_ends(gc, N, n):
    rs, seen, words, stale = random_case(3000 + n, 2, N, 1, n, density=0.3)
    bits = torch.from_numpy(words.view(np.int32)).to(DEV)
    offset = n % 5
    st_d, buf = device_stale(stale, offset)
    ws = torch.empty(gc.gc_coverage_workspace_bytes(), dtype=torch.uint8, device=DEV)
    sets = [[0, 1], [2], [1, 2]] if N == 3 else [sorted(rs.choice(N, 3, replace=False).tolist()) for _ in range(6)]
    sets = [s if len(s) == len(sets[0]) else s * len(sets[0]) for s in sets]
    st_o = stale
    for A, R in (([1], 1), ([0, 2], 2)):
        stats = gc.gc_coverage_update(bits, st_d, A, R)
        st_o, stats_o = oracle.coverage_update(st_o, seen, A, R)
        np.testing.assert_array_equal(stats.cpu().numpy().view(np.uint32), stats_o)
        stats, sel = gc.gc_coverage_update_select(bits, st_d, A, R, 2, workspace=ws)
        st_o, stats_o = oracle.coverage_update(st_o, seen, A, R)
        np.testing.assert_array_equal(stats.cpu().numpy().view(np.uint32), stats_o)
        assert sel.cpu().tolist() == oracle.coverage_select(st_o, seen, 2)
        stats, sc = gc.gc_coverage_update_score(bits, st_d, [2], R, sets, workspace=ws)
        st_o, stats_o = oracle.coverage_update(st_o, seen, [2], R)
        np.testing.assert_array_equal(stats.cpu().numpy().view(np.uint32), stats_o)
        np.testing.assert_array_equal(sc.cpu().numpy().view(np.uint64), oracle.coverage_score(st_o, seen, sets))
        np.testing.assert_array_equal(st_d.cpu().numpy(), st_o)
    buf[offset:offset + stale.size] = 0
    assert not buf.any()


@pytest.mark.parametrize("N,B,H,W", [(13, 2, 9, 9), (64, 9, 30, 41), (13, 85, 3, 683)])
def test_scores_of_few_sets(gc, N, B, H, W):
    rs, seen, words, stale = random_case(4000 + N, B, N, H, W, density=0.2)
    bits = torch.from_numpy(words.view(np.int32)).to(DEV)
    st_d, _ = device_stale(stale, 3)
    ws = torch.empty(gc.gc_coverage_workspace_bytes(), dtype=torch.uint8, device=DEV)
    st_o = stale
    for M, a in ((1, 1), (2, 2), (3, 1), (9, 3), (64, 4)):
        ws.fill_(255)
        sets = [sorted(rs.choice(N - 2, a, replace=False).tolist()) for _ in range(M)]
        A = [N - 1] if M % 2 else [N - 2, 0]
        stats, sc = gc.gc_coverage_update_score(bits, st_d, A, 2, sets, workspace=ws)
        st_o, stats_o = oracle.coverage_update(st_o, seen, A, 2)
        want = oracle.coverage_score(st_o, seen, sets)
        np.testing.assert_array_equal(st_d.cpu().numpy(), st_o)
        np.testing.assert_array_equal(stats.cpu().numpy().view(np.uint32), stats_o)
        np.testing.assert_array_equal(sc.cpu().numpy().view(np.uint64), want)
        ws.fill_(255)
        sc = gc.gc_coverage_score(bits, st_d, sets, workspace=ws)
        np.testing.assert_array_equal(sc.cpu().numpy().view(np.uint64), want)
