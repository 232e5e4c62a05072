"""Short captures: pattern counts taken inside the prep kernel (up to 832 tokens), and query tiles inside the true-mask
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


# rows read 256 keys to a segment and eight segments to a pass: captures around both, rows that end within a lane's four keys
@pytest.mark.parametrize("L", [132, 252, 256, 260, 508, 516, 2044, 2048, 2052, 2308])
@pytest.mark.parametrize("tau", [0.02, -1.0])
def test_true_mask_of_rows(L, tau):
    A = synth_map(np.random.default_rng(L), 2, L)
    A[0, L // 2, ::3] = np.nan
    A[1, L - 1, ::5] = np.inf
    m = B.build_mask(mode=B.DAM_FROM_ATTN_MAP, H=2, L=L, S=L, lam=0.5, eps=1e-8, tau=tau, mu=0.3, attn_sum=torch.from_numpy(A).cuda(),
                     blocks=False)
    art = oracle.derive(A, None, 0.5, 1e-8, tau, 0.3)
    assert np.array_equal(u64(m.true_bits), pack_rows_u64(art.true_mask))


# captures whose true mask the prep kernel makes itself (up to 128 tokens), maps of any alignment, values that no threshold takes
@pytest.mark.parametrize("L", [1, 3, 62, 64, 65, 127, 128, 129])
@pytest.mark.parametrize("shift", [0, 1])
def test_true_mask_of_short_maps(L, shift):
    A = synth_map(np.random.default_rng(L), 3, L)
    A[1, L // 2] = np.nan
    A[2, L - 1, 0] = np.inf
    room = torch.empty(A.size + shift, device="cuda")
    room[shift:] = torch.from_numpy(A.ravel()).cuda()
    m = B.build_mask(mode=B.DAM_FROM_ATTN_MAP, H=3, L=L, S=L, lam=0.5, eps=1e-8, tau=0.02, mu=0.3, attn_sum=room[shift:].view(A.shape),
                     blocks=False)
    art = oracle.derive(A, None, 0.5, 1e-8, 0.02, 0.3)
    assert np.array_equal(u64(m.true_bits), pack_rows_u64(art.true_mask))
    for name in ("diag_cnt", "vert_cnt", "diag_flag", "vert_flag"):
        assert np.array_equal(getattr(m, name).cpu().numpy(), getattr(art, name)), name


# tiles that are full by columns and diagonals together: the one unmatched offset meets matched columns only (its tiles' first
# column), or misses one by a column
@pytest.mark.parametrize("T", [64, 128])
@pytest.mark.parametrize("S", [1024, 1100, 3072])  # scanned in the prep kernel, and by a launch
def test_full_tiles_of_columns_and_diagonals(S, T):
    d, v = (np.zeros((3, S), np.uint8) for _ in range(2))
    d[:] = 1
    d[:, 2 * T + T - 1] = 0           # of tile distance 2 the last offset: column 0 of the tile alone, in its last row
    d[:, 5 * T] = 0                   # of distance 5 the middle one: every column
    v[0, ::T] = 1
    v[1, 1::T] = 1
    v[2] = 1
    v[2, T + 3] = 0
    art = oracle.from_patterns(d, v)
    m = B.build_mask(mode=B.DAM_FROM_PATTERNS, H=3, L=0, S=S, tile_m=T, tile_n=T, diag_in=torch.from_numpy(d).cuda(),
                     vert_in=torch.from_numpy(v).cuda())
    torch.cuda.synchronize()
    test_gpu_mask.check_against_oracle(art, S, T, T, m, dense=False)
    row_ptr, col, kind = (getattr(m, x).cpu().numpy() for x in ("blk_row_ptr", "blk_col", "blk_kind"))
    full = [{(qt, c) for qt in range(S // T) for c, k in zip(col[row_ptr[h, qt]:row_ptr[h, qt + 1]], kind[row_ptr[h, qt]:row_ptr[h, qt + 1]])
             if k & 1} for h in range(3)]
    assert (2, 0) in full[0] and (2, 0) not in full[1] and (2, 0) in full[2] and (5, 0) in full[2] and (6, 1) not in full[2]


# tiles that are not square have no classes: full by their offsets alone, by their columns alone, by both together, and not for one
# unmatched offset in the middle of a tall tile, which its first and last rows do not meet; in the prep kernel and by a launch
@pytest.mark.parametrize("S,tm,tn", [(1024, 64, 128), (1000, 128, 64), (1024, 256, 64), (2500, 64, 128), (2500, 128, 64), (2500, 64, 256),
                                     (3500, 192, 128), (4500, 256, 128), (4500, 256, 64)])
@pytest.mark.parametrize("L", [0, 100])
def test_full_tiles_that_are_not_square(S, tm, tn, L):
    d, v = (np.zeros((6, S), np.uint8) for _ in range(2))
    d[0] = 1
    d[1, :700] = 1
    d[2] = 1
    d[2, [tm + 31, 2 * tm + tn + 3]] = 0  # their columns all matched ...
    v[2, :S // 2] = 1
    d[3] = d[2]                           # ... but one
    v[3] = v[2]
    v[3, 2 * tn + 5] = 0
    d[4] = 1
    d[4, 70::400] = 0
    v[4, ::7] = 1
    d[5, ::90] = 1
    v[5, 64:600] = 1
    tb, true = None, None
    if L:
        true = np.tril(np.random.default_rng(S).random((6, L, L)) < 0.5)
        tb = torch.from_numpy(pack_rows_u64(true).view(np.int64)).cuda()
    art = oracle.from_patterns(d, v, true)
    m = B.build_mask(mode=B.DAM_FROM_PATTERNS, H=6, L=L, S=S, tile_m=tm, tile_n=tn, diag_in=torch.from_numpy(d).cuda(),
                     vert_in=torch.from_numpy(v).cuda(), true_bits=tb)
    torch.cuda.synchronize()
    test_gpu_mask.check_against_oracle(art, S, tm, tn, m, dense=False)
    n_full = [int((m.blk_kind[m.blk_row_ptr[h, 0]:m.blk_row_ptr[h, -1]] & 1).sum()) for h in range(6)]
    assert n_full[0] > n_full[2] > n_full[3] > 0 and n_full[1] > 0 and n_full[5] > 0


# one query tile, the most and one more than the prep kernel scans itself; ragged, inside and beyond the true-mask block
@pytest.mark.parametrize("S,tm,tn,L", [(60, 64, 64, 200), (500, 64, 64, 130), (512, 64, 64, 512), (513, 64, 64, 200), (1000, 128, 64, 300),
                                       (1024, 128, 128, 200), (1025, 128, 128, 200), (700, 256, 64, 64), (1024, 64, 64, 128),
                                       (1025, 64, 64, 129), (2048, 128, 128, 100), (2060, 128, 128, 300)])
def test_scan_inside_the_prep_kernel(S, tm, tn, L):
    run_from_map(synth_map(np.random.default_rng(S), 3, L), None, S, tm, tn, 0.5, 1e-8, 0.02, 0.4)
    if S > tm:
        test_gpu_mask.test_gathered_column_tiles_match_oracle(S, tm, tn, min(L, S // 2))


# the same from patterns alone
@pytest.mark.parametrize("S", [440, 448, 500, 512, 520, 1000, 1024, 1030])
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
