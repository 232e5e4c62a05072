"""Block index of rows of tiles that span several occupancy words (64 tiles each): words that no matched diagonal or column
reaches are passed over by the scan and by the fill, the diagonal tile and gathered tiles beyond every matched diagonal are
decided without looking at their entries. Bit for bit against the oracle, in the plain and in the gathered layout."""
import numpy as np
import pytest
import torch

import oracle
from dam_testlib import pack_rows_u64
from paper_2506_11104_amd import binding as B
from test_gpu_mask import check_against_oracle, check_gathered

pytestmark = pytest.mark.gpu


def patterns(S):
    rng = np.random.default_rng(S)
    d, v = (np.zeros((8, S), np.uint8) for _ in range(2))
    d[0, :40] = 1                                       # a window alone: one word per row of tiles
    d[1, :40] = 1                                       # ... sinks
    v[1, :4] = 1
    d[2, 64] = 1                                        # nothing on the diagonal tile's main diagonal, columns in the middle word
    v[2, [4500, 4600]] = 1
    v[3, rng.choice(S, 200, replace=False)] = 1         # columns only, the last gathered tile incomplete
    d[4, [0, 63, 127, 4096 + 63, 4096 + 64]] = 1        # the reach ends at a word's edge
    v[4, rng.choice(S, 64, replace=False)] = 1          # one complete gathered tile (of 64) and no more
    d[5, S - 1] = 1                                     # the farthest diagonal of all, and nothing else
    d[7, 0] = 1                                         # (head 6: nothing at all) the main diagonal
    v[7, rng.choice(S, 700, replace=False)] = 1
    return d, v


# one, two, three and four words; whole rows of tiles and a ragged last one; a true-mask block that ends inside a tile row;
# tiles of two words (128) and of unequal sides, which have no classes
@pytest.mark.parametrize("S,tm,tn,L", [(4096, 64, 64, 0), (8192, 64, 64, 0), (8256, 64, 64, 100), (12290, 64, 64, 64), (12352, 64, 64, 0),
                                       (16640, 128, 128, 0), (16700, 128, 128, 130), (8300, 128, 64, 0)])
def test_words_and_tiles_that_no_diagonal_reaches(S, tm, tn, L):
    d, v = patterns(max(S, 8192))
    d, v = np.ascontiguousarray(d[:, :S]), np.ascontiguousarray(v[:, :S])
    rng = np.random.default_rng(L)
    t = (rng.random((8, L, L)) < 0.3).astype(np.uint8) * np.tril(np.ones((L, L), np.uint8)) if L else None
    art = oracle.from_patterns(d, v, t)
    tb = torch.from_numpy(pack_rows_u64(t).view(np.int64)).cuda() if L else None
    d_in, v_in = torch.from_numpy(d).cuda(), torch.from_numpy(v).cuda()

    def build(flags):
        m = B.build_mask(mode=B.DAM_FROM_PATTERNS, H=8, L=L, S=S, tile_m=tm, tile_n=tn, diag_in=d_in, vert_in=v_in, true_bits=tb,
                         flags=flags)
        torch.cuda.synchronize()
        return m

    check_against_oracle(art, S, tm, tn, build(0), dense=False)
    check_gathered(art, S, tm, tn, build(B.DAM_MASK_GATHER_COLUMNS))
    check_gathered(art, S, tm, tn, build(B.DAM_MASK_GATHER_COLUMNS | B.DAM_MASK_SKIP_FULL_TILE_BITS), skip_full=True)


# more workgroups than a row of the grid holds (16384): every map the same as in a build of eight
@pytest.mark.parametrize("L", [0, 130])
def test_maps_beyond_the_first_row_of_the_grid(L):
    S, H = 1000, 4200
    d, v = (np.zeros((8, S), np.uint8) for _ in range(2))
    rng = np.random.default_rng(L + 1)
    for h in range(8):
        d[h, :1 + 9 * h] = 1
        v[h, rng.choice(S, 3 * h, replace=False)] = 1
    t = (rng.random((8, L, L)) < 0.3).astype(np.uint8) * np.tril(np.ones((L, L), np.uint8)) if L else None

    def build(copies):
        tb = torch.from_numpy(pack_rows_u64(t).view(np.int64)).cuda().repeat(copies, 1, 1) if L else None
        m = B.build_mask(mode=B.DAM_FROM_PATTERNS, H=8 * copies, L=L, S=S, tile_m=64, tile_n=64, diag_in=torch.from_numpy(d).cuda().repeat(copies, 1),
                         vert_in=torch.from_numpy(v).cuda().repeat(copies, 1), true_bits=tb)
        torch.cuda.synchronize()
        return m

    few, many = build(1), build(H // 8)
    check_against_oracle(oracle.from_patterns(d, v, t), S, 64, 64, few, dense=False)
    n = few.n_tiles
    assert many.n_tiles == n * (H // 8)
    ptr = many.blk_row_ptr.view(H // 8, 8, -1) - n * torch.arange(H // 8, device="cuda", dtype=torch.int32)[:, None, None]
    assert torch.equal(ptr, few.blk_row_ptr[None].expand_as(ptr))
    for name in ("blk_col", "blk_kind", "tile_bits"):
        got, want = getattr(many, name).view(H // 8, n, -1), getattr(few, name).view(1, n, -1)
        assert torch.equal(got, want.expand_as(got)), name
