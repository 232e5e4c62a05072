"""The list of a head's matched columns (gathered layout) and the flags it comes from: words of the column set with none, one, two
and all of their columns, rows of flags of every alignment and of fewer than 16 bytes, more than 1024 words. Whole numbers."""
import numpy as np
import pytest
import torch

from paper_2506_11104_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [1, 15, 16, 17, 63, 65, 1000, 1024, 4103, 65536, 66001, 131072])
def test_matched_columns_in_ascending_order(S):
    rng = np.random.default_rng(S)
    H = 5
    d, v = (np.zeros((H, S), np.uint8) for _ in range(2))
    d[:, 0] = 1
    v[0] = 1                                                       # every word full
    v[1, ::64] = 7                                                 # one of each word (any value but zero is a match)
    v[2, ::64], v[2, 63::64] = 128, 255                            # two, the first and the last
    v[3, rng.random(S) < 0.05] = 1                                 # some of each
    v[3, S // 2:S // 2 + 200] = 1
    m = B.build_mask(mode=B.DAM_FROM_PATTERNS, H=H, L=0, S=S, diag_in=torch.from_numpy(d).cuda(), vert_in=torch.from_numpy(v).cuda(),
                     flags=B.DAM_MASK_GATHER_COLUMNS | B.DAM_MASK_SKIP_FULL_TILE_BITS)
    torch.cuda.synchronize()
    got, cnt = m.gather_idx.cpu().numpy().reshape(H, -1), m.gather_cnt.cpu().numpy()
    for h in range(H):
        want = np.nonzero(v[h])[0]
        assert cnt[h] == len(want)
        assert np.array_equal(got[h, :len(want)], want) and (got[h, len(want):] == -1).all()
