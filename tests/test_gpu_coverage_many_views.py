"""The schedule's calls with more than twelve views, where one launch runs per
greedy round: view counts on both sides of each kernel variant's bound (16 and
32 views per four waves; 64 in all), rows shorter than a pair word, rows that
end inside a word and inside an item of 64 words, staleness at every byte
offset, many more items than blocks; bit-exact against the oracle, whatever
the workspace held."""
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


@pytest.mark.parametrize("N,B,H,W,offset", [
    (13, 1, 1, 1, 0), (16, 2, 3, 11, 1), (17, 1, 33, 63, 2), (20, 2, 95, 97, 3), (32, 1, 64, 32, 0), (33, 1, 45, 46, 5),
    (64, 1, 13, 17, 7), (64, 2, 67, 91, 4), (14, 4, 128, 128, 16)])
def test_update_select_score_many_views(gc, N, B, H, W, offset):
    rs, seen, words, stale = random_case(1000 + N + H, B, N, H, W, density=0.25)
    for u in range(N):   # a view's own row is its producer's to leave as it is
        words[u, :, u] = rs.integers(0, 2**32, words[u, :, u].shape, dtype=np.uint64).astype(np.uint32)
    bits = torch.from_numpy(words.view(np.int32)).to(DEV)
    st_d, buf = device_stale(stale, offset)
    ws = torch.empty(gc.gc_coverage_workspace_bytes(), dtype=torch.uint8, device=DEV)
    st_o = stale
    pick = lambda n: sorted(rs.choice(N, n, replace=False).tolist())  # noqa: E731
    for i, (A, R, a, n_forced) in enumerate([(pick(3), 1, 1, 0), (pick(5), 2, 8, 2), (list(range(N)), 254, 5, 0),
                                             (pick(1), 300, 4, 4), (pick(2), 3, 3, 1)]):
        ws.copy_(torch.randint(0, 256, ws.shape, dtype=torch.uint8, generator=torch.Generator().manual_seed(i)))
        forced = pick(n_forced) if n_forced else []
        sets = [pick(a) for _ in range(64 if i == 1 else 5)]
        st_o, stats_o = oracle.coverage_update(st_o, seen, A, R)
        if i % 2 == 0:
            stats, sel = gc.gc_coverage_update_select(bits, st_d, A, R, a, forced=forced, workspace=ws)
            sc = gc.gc_coverage_score(bits, st_d, sets, workspace=ws)
        else:
            stats, sc = gc.gc_coverage_update_score(bits, st_d, A, R, sets, workspace=ws)
            sel = gc.gc_coverage_select(bits, st_d, a, forced=forced, workspace=ws)
        np.testing.assert_array_equal(st_d.cpu().numpy(), st_o)
        np.testing.assert_array_equal(stats.cpu().numpy().view(np.uint32), stats_o)
        assert sel.cpu().tolist() == oracle.coverage_select(st_o, seen, a, forced)
        np.testing.assert_array_equal(sc.cpu().numpy().view(np.uint64), oracle.coverage_score(st_o, seen, sets))
    n = stale.size
    left = buf.clone()
    left[offset:offset + n] = 0
    assert not left.any()   # nothing written around the staleness


@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 1024, 4093])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_initial_staleness(gc, n, offset):
    """0 for foreground and 255 for background, whatever the count leaves for
    the last thread and wherever the bytes start."""
    rs = np.random.default_rng(n)
    P = rs.standard_normal((1, 1, 1, n, 3)).astype(np.float32)
    P[0, 0, 0, rs.random(n) < 0.5, 1] = np.nan
    P[0, 0, 0, rs.random(n) < 0.1, 2] = -np.inf
    buf = torch.full((n + 16,), 7, dtype=torch.uint8, device=DEV)
    out = buf[offset:offset + n].view(1, 1, 1, n)
    gc.gc_coverage_init(torch.from_numpy(P).to(DEV), out=out)
    want = np.full(n + 16, 7, np.uint8)
    want[offset:offset + n] = np.where(np.isfinite(P[0, 0, 0]).all(-1), 0, 255)
    np.testing.assert_array_equal(buf.cpu().numpy(), want)
