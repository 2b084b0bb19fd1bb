"""The area downsample (every staged factor, a factor without one; the factors
with a variant for small inputs also around its bound) and the bounding box,
bit-exact against the oracle, at the sizes where their launches change: pixel
counts around a wave's 64 and a block's 256, rows shorter than a wave and rows
that a wave crosses, several small maps in one wave; assets up to and above the
one-block bound of the box, sample counts that leave threads without a sample,
an asset without foreground, infinite positions."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def gc():
    import paper_2608_13255_amd as gc
    return gc


def render(rs, shape):
    P = rs.standard_normal(shape + (3,)).astype(np.float32)
    P[rs.random(shape) < 0.45] = np.nan
    P[..., 0][rs.random(shape) < 0.02] = np.inf
    return P


@pytest.mark.parametrize("f", [2, 3, 4, 6, 8, 16, 1, 5])
@pytest.mark.parametrize("n,H,W", [(1, 1, 1), (2, 1, 63), (1, 5, 13), (3, 8, 8), (1, 3, 65), (2, 16, 16), (7, 3, 5),
                                   (1, 1, 257), (2, 33, 31)])
def test_downsample_matches_oracle(gc, f, n, H, W):
    rs = np.random.default_rng(f * 1000 + H * 10 + W)
    hi = render(rs, (1, n, H * f, W * f))
    got = gc.gc_posmap_downsample(torch.from_numpy(hi).to(DEV), f).cpu().numpy()
    want = oracle.downsample(hi, f)
    np.testing.assert_array_equal(got.view(np.int32), want.view(np.int32))


@pytest.mark.parametrize("f", [4, 8])
@pytest.mark.parametrize("H,W", [(1, 63), (5, 13), (3, 65), (8, 8), (1, 257), (33, 31)])
@pytest.mark.parametrize("more", [0, 1])
def test_downsample_around_the_small_bound(gc, f, H, W, more):
    """The last input within the 48 MiB of the variant for small ones, and one map more."""
    n = (48 << 20) // (H * W * f * f * 12) + more
    rs = np.random.default_rng(f * 1000 + H * 10 + W)
    one = render(rs, (1, 53, H * f, W * f))
    hi = np.tile(one, (1, n // 53 + 1, 1, 1, 1))[:, :n]
    got = gc.gc_posmap_downsample(torch.from_numpy(hi).to(DEV), f).cpu().numpy()
    want = np.tile(oracle.downsample(one, f), (1, n // 53 + 1, 1, 1, 1))[:, :n]
    np.testing.assert_array_equal(got.view(np.int32), want.view(np.int32))


@pytest.mark.parametrize("B,N,H,W", [(1, 1, 1, 1), (3, 1, 1, 1023), (2, 1, 31, 33), (2, 2, 128, 128), (2, 1, 1, 4094),
                                     (3, 9, 61, 60), (1, 1, 4094, 8), (1, 1, 4094, 9), (5, 12, 97, 91), (1, 64, 130, 130)])
def test_bbox_matches_oracle(gc, B, N, H, W):
    rs = np.random.default_rng(B + N + H + W)
    P = render(rs, (B, N, H, W))
    if B > 1:
        P[B - 1] = np.nan
    want = np.zeros((B, 8), np.float32)
    o = oracle.bbox(P, 0.03)
    want[:, :o.shape[1]] = o
    Pd = torch.from_numpy(P).to(DEV)
    for _ in range(3):
        out = torch.full((B, 8), 7.0, device=DEV)
        got = gc.gc_posmap_bbox(Pd, 0.03, bbox=out).cpu().numpy()
        np.testing.assert_array_equal(got.view(np.int32), want.view(np.int32))
