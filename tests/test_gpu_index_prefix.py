"""Both token indexes (bits, list, count; whole numbers, bit-exact against
their definition) where the scatter pass finds its block's place in the list:
bands and tiles cut by the grid's edges, blocks of 1024 list positions that
start inside a tile, views that start inside a bit word, very long and very
narrow grids, no listed token and nothing but listed tokens, and token counts
at and above the bound from which a scan pass gives the chunks' offsets."""
import numpy as np
import pytest
import torch

from conftest import listed_in_tile_order

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = [(1, 1, 1), (3, 1, 700), (2, 700, 1), (5, 17, 33), (7, 31, 49), (1, 3, 4094), (1, 4094, 3), (9, 75, 101)]
LARGE = [(64, 512, 512), (66, 511, 509)]   # 16384 chunks and a few more


@pytest.fixture(scope="module")
def gc():
    import paper_2608_13255_amd as gc
    return gc


def check_bits(words, flags):
    un = np.unpackbits(np.ascontiguousarray(words.cpu().numpy().view(np.uint32)).view(np.uint8), bitorder="little")
    np.testing.assert_array_equal(un[:flags.size].astype(bool), flags)
    assert not un[flags.size:].any()


@pytest.mark.parametrize("n_views,H,W,density", [(*s, d) for s in SHAPES for d in (0.0, 0.3, 1.0)] +
                         [(*s, 0.3) for s in LARGE])
def test_indexes_match_their_definition(gc, n_views, H, W, density):
    rs = np.random.default_rng(n_views * 7919 + H * 31 + W)
    n = n_views * H * W
    a = 1 if n > 1 << 20 else int(rs.integers(1, 9))
    flags = rs.random(n) < density
    want = listed_in_tile_order(flags, H, W)
    corr = np.zeros((n, a), np.int32)
    corr[np.arange(n), rs.integers(0, a, n)] = flags * np.int32(0x01001001)
    cd = torch.from_numpy(corr.reshape(1, n_views, H, W, a)).to(DEV)
    for idx in (gc.gc_index_correspondence(cd), gc.gc_index_correspondence_noalloc(cd)):
        assert idx.n_vis == want.size
        np.testing.assert_array_equal(idx.vis_list.cpu().numpy()[:want.size], want)
        check_bits(idx.vis_bits, flags)
    pos = rs.uniform(-1, 1, (n, 3)).astype(np.float32)
    pos[np.flatnonzero(~flags), rs.integers(0, 3, int((~flags).sum()))] = np.nan
    fg = gc.gc_index_foreground(torch.from_numpy(pos.reshape(n_views, H, W, 3)).to(DEV))
    assert fg.n_fg == want.size
    recs = fg.fg_recs.cpu().numpy()[:want.size]
    np.testing.assert_array_equal(recs[:, 0], want)
    np.testing.assert_array_equal(recs[:, 1:], pos[want].view(np.int32))
    check_bits(fg.fg_bits, flags)
