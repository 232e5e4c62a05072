"""bf16 prefill, more items than the chip has workgroups: taken by length (the workspace has room for the order) or by number
(a workspace without that room), every row comes out the same; and the order that was taken, which the workspace still holds,
is one of every item, longest first."""
import numpy as np
import pytest
import torch

from paper_2506_11104_amd import binding as B

pytestmark = pytest.mark.gpu
ORDER = 8 * 512 * 16  # eight queues of up to 512 items, 16 bytes each
GROUP, BINS = 192, 512  # pairs go in groups of that many items or more; lengths are told apart below 512 / groups


def check_order(order, mask, batch, hq, hkv, S):
    """{item, first tile, end} per place of a queue: every item once, with its own tiles, groups of pairs one after the other,
    no item in front of a longer one of its group."""
    row_ptr, kind = mask.blk_row_ptr.cpu().numpy().astype(np.int64), mask.blk_kind.cpu().numpy()
    blocks_before = np.concatenate([[0], np.cumsum(sum((kind >> b) & 1 for b in range(1, 5)).astype(np.int64))])
    G, nQt, pairs = hq // hkv, (S + 127) // 128, batch * hkv
    per_pair, even = G * nQt, pairs % 8 == 0
    group_pairs = -(-GROUP // per_pair)
    groups = max(1, pairs // 8 // group_pairs) if even else 1
    for qu in range(8):
        n = pairs // 8 * per_pair if even else (pairs * per_pair - qu + 7) // 8
        item, t0, t1 = order[qu, :n, :3].T.astype(np.int64)
        assert np.array_equal(np.sort(item), np.arange(n))
        pair, within = (item // per_pair * 8 + qu, item % per_pair) if even else ((item * 8 + qu) % pairs, (item * 8 + qu) // pairs)
        head, qt = pair % hkv * G + within % G, nQt - 1 - within // G
        assert np.array_equal(t0, row_ptr[head, qt]) and np.array_equal(t1, row_ptr[head, qt + 1])
        cut = np.minimum(t1, t0 + 64)
        length = np.minimum(blocks_before[cut] - blocks_before[t0] + 2 * (t1 - cut), BINS // groups - 1)
        group = np.minimum(item // (group_pairs * per_pair), groups - 1)
        assert (np.diff(group) >= 0).all() and (np.diff(length)[np.diff(group) == 0] <= 0).all()
        assert len(np.unique(length)) > 3


@pytest.mark.parametrize("shift", [0, 1, 2, 3])  # of the tile kinds' first byte from a multiple of four
@pytest.mark.parametrize("batch,hq,hkv,S,flags", [
    (1, 30, 5, 3400, 0),                           # five pairs: every eighth item to a queue, a ragged last tile
    (2, 32, 4, 2176, B.DAM_MASK_GATHER_COLUMNS),   # eight pairs, gathered tiles
    (1, 16, 16, 9000, 0),                          # rows of more than 64 listed tiles
    (8, 32, 8, 2048, 0),                           # 512 items a queue: the longest one put into order
])
def test_the_order_of_the_items_changes_nothing(batch, hq, hkv, S, flags, shift):
    gen = torch.Generator(device="cuda").manual_seed(S)
    rng = np.random.default_rng(S)
    d, v = (np.zeros((hq, S), np.uint8) for _ in range(2))
    for h in range(hq):
        if h % 5:  # (a head without patterns has no listed tiles)
            d[h, : S if h == 1 else 1 + rng.integers(0, 700)] = 1
            v[h, rng.integers(0, S, 12)] = 1
    mask = B.build_mask(mode=B.DAM_FROM_PATTERNS, H=hq, L=0, S=S, diag_in=torch.from_numpy(d).cuda(), vert_in=torch.from_numpy(v).cuda(),
                        flags=flags)
    kinds = torch.full((mask.blk_kind.numel() + shift,), 0xFF, dtype=torch.uint8, device="cuda")
    kinds[shift:] = mask.blk_kind
    mask.blk_kind = kinds[shift:]
    q, k, v_ = (torch.randn((batch, h, S, 128), generator=gen, device="cuda", dtype=torch.bfloat16) for h in (hq, hkv, hkv))
    ws = B.prefill_workspace(B.attn_params(q, k, v_, torch.empty_like(q), 128, 128, gather_rows=mask.gather_rows), "cuda")
    got = []
    for room in (ws, ws[:-ORDER]):
        ws.fill_(0xFF)
        out = torch.full_like(q, 7.0)
        got.append(B.dam_sparse_attn_prefill(q, k, v_, mask, out=out, ws=room, want_lse=True))
        if room is ws:
            check_order(ws[-ORDER:].cpu().numpy().view(np.int32).reshape(8, 512, 4), mask, batch, hq, hkv, S)
    with pytest.raises(RuntimeError):
        B.dam_sparse_attn_prefill(q, k, v_, mask, ws=ws[:-ORDER - 256])
    torch.cuda.synchronize()
    (o1, l1), (o2, l2) = got
    assert torch.equal(o1, o2) and torch.equal(l1, l2)
    assert not bool((o1 == 7.0).all(-1).any())


def test_a_workspace_of_a_larger_batch_has_room_for_the_order():
    """Queues of more than 512 items are not sorted, but their workspace serves a smaller batch, whose queues are."""
    hq, hkv, S = 32, 8, 2176
    gen = torch.Generator(device="cuda").manual_seed(1)
    rng = np.random.default_rng(1)
    d = np.zeros((hq, S), np.uint8)
    for h in range(hq):
        d[h, : 1 + rng.integers(0, 700)] = 1
    mask = B.build_mask(mode=B.DAM_FROM_PATTERNS, H=hq, L=0, S=S, diag_in=torch.from_numpy(d).cuda(), vert_in=torch.zeros_like(torch.from_numpy(d)).cuda())
    q, k, v = (torch.randn((8, h, S, 128), generator=gen, device="cuda", dtype=torch.bfloat16) for h in (hq, hkv, hkv))
    ws, small = (B.prefill_workspace(B.attn_params(q[:b], k[:b], v[:b], torch.empty_like(q[:b]), 128, 128), "cuda") for b in (8, 2))
    assert small.numel() <= ws.numel()
    ws.fill_(0xFF)
    out = B.dam_sparse_attn_prefill(q, k, v, mask, ws=ws)
    torch.cuda.synchronize()
    assert bool((ws[-ORDER:] == 0xFF).all())
    few = B.dam_sparse_attn_prefill(q[:2], k[:2], v[:2], mask, ws=ws)
    check_order(ws[small.numel() - ORDER:small.numel()].cpu().numpy().view(np.int32).reshape(8, 512, 4), mask, 2, hq, hkv, S)
    assert torch.equal(few, out[:2])
