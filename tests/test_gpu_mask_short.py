"""Short captures: pattern counts taken inside the prep kernel (up to 768 tokens, 832 where nothing follows them), and query tiles inside the true-mask
block, whose tiles the scan looks at four at a time. Bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from dam_testlib import pack_rows_u64, u64
from paper_2506_11104_amd import binding as B
import test_gpu_mask
from test_gpu_mask import run_from_map, synth_map

pytestmark = pytest.mark.gpu


# one word, its neighbours, whole and ragged chunks, one chunk more and less than a round of waves
@pytest.mark.parametrize("L", [1, 2, 63, 64, 65, 200, 512, 1023, 1024, 1025])
@pytest.mark.parametrize("mu", [0.0, 0.3, 1.0])
def test_pattern_counts_of_short_captures(L, mu):
    A = synth_map(np.random.default_rng(L), 2, L)
    run_from_map(A, None, L + 70, 64, 64, 0.5, 1e-8, 0.02, mu, dense=False)


@pytest.mark.parametrize("L", [96, 1000])
def test_pattern_counts_without_a_block_index(L):
    A = synth_map(np.random.default_rng(L), 3, L)
    art = oracle.derive(A, None, 0.5, 1e-8, 0.02, 0.3)
    mask = B.build_mask(mode=B.DAM_FROM_ATTN_MAP, H=3, L=L, S=L, lam=0.5, eps=1e-8, tau=0.02, mu=0.3,
                        attn_sum=torch.from_numpy(A).cuda(), blocks=False)
    assert np.array_equal(u64(mask.true_bits), pack_rows_u64(art.true_mask))
    for name in ("diag_cnt", "vert_cnt", "diag_flag", "vert_flag"):
        assert np.array_equal(getattr(mask, name).cpu().numpy(), getattr(art, name)), name


# tiles of 1, 2, 3 and 4 words per lane and one of 16 (the general form); 9 tiles are two steps of four and one more
@pytest.mark.parametrize("tm,tn", [(64, 64), (128, 64), (192, 64), (128, 128), (64, 256), (256, 64), (256, 256)])
@pytest.mark.parametrize("S", [575, 576, 700])
def test_tiles_of_the_true_mask_block(tm, tn, S):
    A = synth_map(np.random.default_rng(S), 2, 576)
    A[0, :300, :300] = np.tril(np.full((300, 300), 0.5, np.float32))  # full tiles
    A[1, 128:256, :128] = 0.0                                         # empty ones
    run_from_map(A, None, S, tm, tn, 0.5, 1e-8, 0.02, 0.8)


# captures whose patterns are counted with nothing else to do: in the prep kernel up to 832 tokens, in chunks of 128 rows beyond,
# with whole and ragged last chunks, for few and for many maps
@pytest.mark.parametrize("L,copies", [(768, 1), (769, 1), (800, 30), (831, 1), (832, 1), (833, 1), (895, 1), (896, 1), (897, 1), (1024, 1), (897, 23),
                                      (897, 24), (1024, 24)])
def test_pattern_counts_alone_on_both_sides_of_the_line(L, copies):
    A = synth_map(np.random.default_rng(L + copies), 2, L)
    art = oracle.derive(A, None, 0.5, 1e-8, 0.02, 0.3)
    a_dev = torch.from_numpy(A).cuda().repeat(copies, 1, 1)
    mask = B.build_mask(mode=B.DAM_FROM_ATTN_MAP, H=2 * copies, L=L, S=L, lam=0.5, eps=1e-8, tau=0.02, mu=0.3, attn_sum=a_dev,
                        blocks=False)
    for name in ("diag_cnt", "vert_cnt", "diag_flag", "vert_flag"):
        assert np.array_equal(getattr(mask, name).cpu().numpy(), np.tile(getattr(art, name), (copies, 1))), name


# one query tile, the most and one more than the prep kernel scans itself; ragged, inside and beyond the true-mask block
@pytest.mark.parametrize("S,tm,tn,L", [(60, 64, 64, 200), (500, 64, 64, 130), (512, 64, 64, 512), (513, 64, 64, 200), (1000, 128, 64, 300),
                                       (1024, 128, 128, 200), (1025, 128, 128, 200), (700, 256, 64, 64)])
def test_scan_inside_the_prep_kernel(S, tm, tn, L):
    run_from_map(synth_map(np.random.default_rng(S), 3, L), None, S, tm, tn, 0.5, 1e-8, 0.02, 0.4)
    if S > tm:
        test_gpu_mask.test_gathered_column_tiles_match_oracle(S, tm, tn, min(L, S // 2))


# the same from patterns alone, whose line in the plain layout is seven query tiles for a ragged length
@pytest.mark.parametrize("S", [440, 448, 500, 512, 520])
def test_scan_of_patterns_inside_the_prep_kernel(S):
    rng = np.random.default_rng(S)
    d, v = (np.zeros((4, S), np.uint8) for _ in range(2))
    for h in range(3):
        d[h, :1 + 60 * h] = 1
        d[h, rng.choice(S, 5, replace=False)] = 1
        v[h, rng.choice(S, 9 * h + 2, replace=False)] = 1
    art = oracle.from_patterns(d, v)
    for flags, check in ((0, lambda m: test_gpu_mask.check_against_oracle(art, S, 64, 64, m, dense=False)),
                         (B.DAM_MASK_GATHER_COLUMNS, lambda m: test_gpu_mask.check_gathered(art, S, 64, 64, m))):
        m = B.build_mask(mode=B.DAM_FROM_PATTERNS, H=4, L=0, S=S, tile_m=64, tile_n=64, diag_in=torch.from_numpy(d).cuda(),
                         vert_in=torch.from_numpy(v).cuda(), flags=flags)
        torch.cuda.synchronize()
        check(m)
