"""The fp32 prefill kernel at the sizes where its tiling can go wrong: 16-row groups, blocks of 16 keys shared by four
waves, 64 listed tiles per segment, work numbering with and without a whole number of heads per XCD.
Tolerance: sums of at most S products of O(1) values in fp32 against the fp64 oracle, S 2^-24 times a few: 2e-5."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_11104_amd import binding as B
from test_gpu_prefill import gpu_mask_from_art

pytestmark = pytest.mark.gpu
TOL = 2e-5


def inputs(Hq, Hkv, S, d, seed):
    rng = np.random.default_rng(seed)
    Q, K, V = (rng.standard_normal((h, S, d)).astype(np.float32) for h in (Hq, Hkv, Hkv))
    dflag, vflag = np.zeros((Hq, S), np.uint8), np.zeros((Hq, S), np.uint8)
    dflag[0] = 1                                    # dense causal
    for h in range(1, Hq):
        dflag[h, : 1 + 7 * h % max(1, S)] = 1
        vflag[h, :: 19 + h] = 1
    return Q, K, V, oracle.from_patterns(dflag, vflag)


def run(Q, K, V, mask):
    t = lambda x: torch.from_numpy(x)[None].cuda()
    out, lse = B.dam_sparse_attn_prefill(t(Q), t(K), t(V), mask, want_lse=True)
    return out[0].cpu().numpy(), lse[0].cpu().numpy()


@pytest.mark.parametrize("Hq,Hkv,S,d,tile,flags", [
    (2, 1, 1, 64, 64, 0), (2, 2, 15, 128, 128, 0), (4, 2, 17, 64, 128, 0), (2, 1, 65, 128, 64, 0),
    (8, 8, 130, 64, 64, 0), (16, 8, 259, 128, 128, B.DAM_MASK_GATHER_COLUMNS), (3, 3, 640, 64, 64, B.DAM_MASK_GATHER_COLUMNS),
    (12, 4, 700, 128, 64, 0), (12, 6, 690, 64, 128, B.DAM_MASK_GATHER_COLUMNS),  # more than 512 workgroups
    (16, 2, 1021, 128, 128, B.DAM_MASK_GATHER_COLUMNS),
    (1, 1, 64 * 66 + 5, 64, 64, 0),                 # more listed tiles in a row than one segment holds
])
def test_edges_of_groups_blocks_and_segments(Hq, Hkv, S, d, tile, flags):
    Q, K, V, art = inputs(Hq, Hkv, S, d, 7 + S)
    mask = gpu_mask_from_art(art, S, tile, tile, flags=flags | B.DAM_MASK_SKIP_FULL_TILE_BITS)
    out, lse = run(Q, K, V, mask)
    O, LSE = oracle.attend_prefill(Q, K, V, art)
    assert np.abs(out - O).max() <= TOL
    assert np.abs(lse - LSE).max() <= TOL


# in few workgroups (one form of the kernel) and in more than 512 of them (whose second form takes such rows again)
@pytest.mark.parametrize("copies,d", [(1, 128), (40, 128), (40, 64)])
def test_a_row_does_not_see_what_it_does_not_keep(copies, d):
    """A NaN and an infinity in V rows reach exactly the query rows that keep those keys."""
    S, far = 200, 70 if d == 128 else 60  # (of 128 dims, one in either half)
    Q, K, V, art = inputs(2, 1, S, d, 5)
    V[0, 37, 3], V[0, 101, far] = np.nan, np.inf
    mask = gpu_mask_from_art(art, S, 64, 64)
    t = lambda x: torch.from_numpy(x)[None].cuda().repeat(copies, 1, 1, 1)
    v = t(V)
    v[1:, 0, 37, 3] = v[1:, 0, 101, far] = 1.0  # (the other sequences' values are finite)
    outs, lses = B.dam_sparse_attn_prefill(t(Q), t(K), v, mask, want_lse=True)
    out = outs[0].cpu().numpy()
    if copies > 1:
        Vf = V.copy()
        Vf[0, 37, 3] = Vf[0, 101, far] = 1.0
        O, LSE = oracle.attend_prefill(Q, K, Vf, art)
        assert np.abs(outs[-1].cpu().numpy() - O).max() <= TOL and np.abs(lses.cpu().numpy() - LSE).max() <= TOL
    i = np.arange(S)
    for h, keeps in ((0, lambda j: i >= j), (1, lambda j: (i >= j) & ((i - j < 8) | (j % 20 == 0)))):
        assert np.array_equal(np.isnan(out[h, :, 3]), keeps(37))
        assert np.array_equal(np.isinf(out[h, :, far]), keeps(101))
        assert np.isfinite(out[h, :, 5]).all()


# the only odd value in one dim, in each quarter of the dims and at their ends: the first form of more than 512 workgroups has to
# notice it wherever it is (a row that does not keep the key would get a NaN from the product with its zero weight)
@pytest.mark.parametrize("d,dim", [(128, 0), (128, 35), (128, 64), (128, 95), (128, 96), (128, 127), (64, 0), (64, 31), (64, 63)])
@pytest.mark.parametrize("value", [np.nan, -np.inf])
def test_one_odd_value_is_noticed_in_any_dim(d, dim, value):
    S = 200
    Q, K, V, art = inputs(2, 1, S, d, 5)
    V[0, 101, dim] = value
    mask = gpu_mask_from_art(art, S, 64, 64)
    t = lambda x: torch.from_numpy(x)[None].cuda().repeat(40, 1, 1, 1)
    out = B.dam_sparse_attn_prefill(t(Q), t(K), t(V), mask)
    i = np.arange(S)
    for h, keeps in ((0, lambda j: i >= j), (1, lambda j: (i >= j) & ((i - j < 8) | (j % 20 == 0)))):
        want = np.zeros((S, d), bool)
        want[:, dim] = keeps(101)
        assert bool((torch.isfinite(out[:, h]) == torch.from_numpy(~want).cuda()).all())


@pytest.mark.parametrize("d", [64, 128])
def test_rows_with_nothing_but_minus_infinity_have_no_value(d):
    """Keys 90 to 129 have logits of -inf: weight 0 beside an ordinary key, whichever comes first; a row that keeps only such
    keys is NaN, as in the oracle, and one that keeps none is zero."""
    S = 200
    Q, K, V, art = inputs(2, 1, S, d, 6)
    Q[:, :, 0], K[0, 90:130, 0] = 1.0, -np.inf
    art.vert_flag[1] = 0
    art.diag_flag[1] = 0
    art.diag_flag[1, 1:4] = 1                       # head 1: rows 93 .. 130 keep three such keys, row 0 none
    out, lse = run(Q, K, V, gpu_mask_from_art(art, S, 64, 64))
    O, LSE = oracle.attend_prefill(Q, K, V, art)
    none = np.arange(S) == 0
    only = (np.arange(S) >= 93) & (np.arange(S) <= 130)
    assert np.isnan(O[1, only]).all() and np.isnan(out[1, only]).all() and (out[1, none] == 0).all()
    assert np.abs(out[0] - O[0]).max() <= TOL and np.abs(out[1, ~only] - O[1, ~only]).max() <= TOL


def test_a_column_list_shorter_than_a_tile():
    """gather_idx of 8 slots per head beside a plain block index (gather_rows 0): no slot is looked up, the list is not read."""
    S = 300
    Q, K, V, art = inputs(4, 2, S, 64, 8)
    mask = gpu_mask_from_art(art, S, 64, 64)
    want, _ = run(Q, K, V, mask)
    mask.gather_idx = torch.full((4, 8), -1, dtype=torch.int32, device="cuda")
    mask.gather_cnt = torch.zeros(4, dtype=torch.int32, device="cuda")
    got, _ = run(Q, K, V, mask)
    assert np.array_equal(got, want)
