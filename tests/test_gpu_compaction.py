"""The kernels that evaluate the operator (the correspondence builder, with
and without counters, and the visibility pairs), at the sizes where a wave of
64 tokens, a chunk of 128 or 256 or a group of 64 compacted foreground tokens
begins or ends: words, pair bits and counters bit-exact against the oracle,
weights within a few float roundings of a quotient (1e-6).  Single assets take
the direct launches, a lane per raster token; the same views in large batches
take those on compacted foreground tokens.  Maps full of foreground, without
any, with one token and with random holes; NaN and infinite positions as
background; pinhole and orthographic cameras in one rig; anchor counts on both
sides of the four- and eight-lane groups; a squared tolerance that overflowed
to infinity, which every finite tap on the grid satisfies."""
import numpy as np
import pytest
import torch

import oracle

from conftest import visible_weights
from test_gpu_limits import sphere_problem
from test_gpu_properties import random_rig

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def gc():
    import paper_2608_13255_amd as gc
    return gc


def problem(seed, N, H, W, fill):
    rs, P, cams = sphere_problem(seed, N, H, W)
    pin = random_rig(rs, N, H, W, True)
    for k in cams:                       # every other camera is a pinhole
        cams[k][0, 1::2] = pin[k][1::2]
    P = P.copy()
    if fill == "all":
        P = np.where(np.isfinite(P), P, rs.uniform(-0.5, 0.5, P.shape).astype(np.float32))
    elif fill == "none":
        P[:] = np.nan
    elif fill == "one":
        keep = P[0, :, H // 2, W // 2].copy()
        P[:] = np.nan
        P[0, :, H // 2, W // 2] = np.where(np.isfinite(keep), keep, 0.1)
    else:
        hole = rs.random(P.shape[:-1]) < 0.3
        P[hole] = np.where(rs.random((int(hole.sum()), 1)) < 0.5, np.float32(np.nan), np.float32(np.inf))
    return rs, P, cams


def device_box(bb):
    full = np.zeros((bb.shape[0], 8), np.float32)
    full[:, :bb.shape[1]] = bb
    return torch.from_numpy(full).to(DEV)


def check_builder(gc, P, cams, bb, anchors, K):
    B, N, H, W = P.shape[:4]
    a = len(anchors)
    corr_o, wts_o, nvis_o = oracle.build(P, cams, anchors, K, bb)
    Pd, cams_d, bbd = torch.from_numpy(P).to(DEV), gc.camera_tensor(cams, DEV), device_box(bb)
    for counted in (False, True):
        stats = torch.full((B, 4), 77, dtype=torch.int32, device=DEV) if counted else None
        corr = torch.full((B, N - a, H, W, a), -1, dtype=torch.int32, device=DEV)
        wts = torch.zeros((B, N - a, H, W, a, K), dtype=torch.float32, device=DEV)
        gc.gc_build_correspondence(Pd, cams_d, anchors, K, bbd, corr=corr, weights=wts, stats=stats)
        np.testing.assert_array_equal(corr.cpu().numpy(), corr_o)
        assert np.abs(visible_weights(corr, wts) - wts_o).max(initial=0.0) <= 1e-6
        if counted:
            targets = [v for v in range(N) if v not in anchors]
            each = tuple(range(1, 5))
            taps = sum(((corr_o >> (24 + k)) & 1).sum(axis=each) for k in range(4))
            want = np.stack([(corr_o != 0).sum(axis=each), (nvis_o > 0).sum(axis=each[:-1]),
                             np.isfinite(P[:, targets]).all(-1).sum(axis=each[:-1]), taps], axis=1)
            np.testing.assert_array_equal(stats.cpu().numpy(), want)


def check_pairs(gc, P, cams, bb):
    B, N, H, W = P.shape[:4]
    pb = gc.gc_coverage_pairs(torch.from_numpy(P).to(DEV), gc.camera_tensor(cams, DEV), device_box(bb),
                              out=torch.full((N, B, N, (H * W + 31) // 32), -1, dtype=torch.int32, device=DEV))
    un = np.unpackbits(pb.cpu().numpy().view(np.uint8), axis=-1, bitorder="little").reshape(N, B, N, -1)
    assert not un[..., H * W:].any()
    np.testing.assert_array_equal(un[..., :H * W].reshape(N, B, N, H, W), oracle.coverage_pairs(P, cams, 4, bb))


def batch(seed, B, N, H, W, fill):
    """B assets with the views of one and holes of their own, the last without any foreground."""
    rs, P, cams = problem(seed, N, H, W, fill)
    P = np.repeat(P, B, axis=0)
    if fill == "holes":
        P[rs.random(P.shape[:-1]) < 0.3] = np.nan
    P[-1] = np.nan
    return rs, P, {k: np.repeat(v, B, axis=0) for k, v in cams.items()}


@pytest.mark.parametrize("N,H,W,a,K,fill", [
    (3, 1, 1, 1, 4, "all"), (3, 1, 63, 2, 4, "all"), (4, 8, 8, 3, 1, "holes"), (4, 5, 13, 4, 4, "all"),
    (5, 15, 17, 4, 4, "holes"), (5, 16, 16, 4, 2, "all"), (6, 257, 1, 5, 4, "all"), (6, 16, 20, 5, 3, "holes"),
    (9, 23, 31, 8, 4, "holes"), (4, 32, 33, 2, 4, "none"), (4, 32, 33, 2, 4, "one"), (9, 33, 32, 1, 4, "all")])
@pytest.mark.parametrize("overflow", [False, True])
def test_builder_and_pairs_match_oracle(gc, N, H, W, a, K, fill, overflow):
    rs, P, cams = problem(7 + N * H + W, N, H, W, fill)
    bb = oracle.bbox(P, 0.05).reshape(1, -1).copy()
    if overflow:
        bb[:, 6] = np.inf
    anchors = sorted(rs.choice(N, a, replace=False).tolist())
    check_builder(gc, P, cams, bb, anchors, K)
    check_pairs(gc, P, cams, bb)


@pytest.mark.parametrize("overflow", [False, True])
@pytest.mark.parametrize("B,N,H,W,fill", [
    # 1024 and 1026 compacted blocks, more than 2048 direct ones
    (256, 4, 1, 63, "all"), (171, 6, 8, 8, "all"), (342, 3, 16, 16, "holes"), (129, 5, 257, 1, "all"),
    (114, 9, 15, 17, "holes"), (65, 8, 16, 20, "one"), (65, 8, 23, 31, "holes"), (55, 13, 33, 32, "all"),
    # 16384 direct blocks of few compacted ones, and some more
    (64, 16, 3, 11, "holes"), (8, 64, 13, 17, "holes"), (9, 64, 16, 16, "all"), (15, 63, 7, 9, "all")])
def test_pairs_of_batches_match_oracle(gc, B, N, H, W, fill, overflow):
    _, P, cams = batch(11 + N * H + W, B, N, H, W, fill)
    bb = oracle.bbox(P, 0.05).copy()
    if overflow:
        bb[::2, 6] = np.inf
    check_pairs(gc, P, cams, bb)


# target tokens up to and above each launch's line: 49,152 with the counters,
# 524,288 (a <= 4) and 786,432 without
@pytest.mark.parametrize("overflow", [False, True])
@pytest.mark.parametrize("B,N,H,W,a,K,fill", [
    (2048, 5, 8, 8, 1, 4, "all"), (2081, 5, 1, 63, 1, 1, "holes"), (683, 8, 8, 16, 2, 4, "all"),
    (241, 12, 257, 1, 3, 2, "holes"), (256, 12, 16, 16, 4, 4, "all"), (197, 12, 19, 19, 4, 3, "holes"),
    (64, 9, 8, 24, 5, 4, "holes"), (66, 9, 11, 17, 5, 4, "all"), (400, 14, 1, 257, 6, 4, "holes"),
    (193, 24, 16, 16, 8, 2, "all"), (120, 32, 17, 16, 8, 4, "one")])
def test_builds_of_batches_match_oracle(gc, B, N, H, W, a, K, fill, overflow):
    rs, P, cams = batch(13 + N * H + W, B, N, H, W, fill)
    bb = oracle.bbox(P, 0.05).copy()
    if overflow:
        bb[::2, 6] = np.inf
    check_builder(gc, P, cams, bb, sorted(rs.choice(N, a, replace=False).tolist()), K)
