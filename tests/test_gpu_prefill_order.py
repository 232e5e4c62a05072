"""bf16 prefill, more items than the chip has workgroups: taken by length (the workspace has room for the order) or by number
(a workspace without that room, as one sized for a larger batch may be), every row comes out the same."""
import numpy as np
import pytest
import torch

from paper_2506_11104_amd import binding as B

pytestmark = pytest.mark.gpu
ORDER = 8 * 512 * 16  # eight queues of up to 512 items, 16 bytes each


@pytest.mark.parametrize("batch,hq,hkv,S,flags", [
    (1, 30, 5, 3400, 0),                           # five pairs: every eighth item to a queue, a ragged last tile
    (2, 32, 4, 2176, B.DAM_MASK_GATHER_COLUMNS),   # eight pairs, gathered tiles
    (1, 16, 16, 9000, 0),                          # rows of more than 64 listed tiles
    (8, 32, 8, 2048, 0),                           # 512 items a queue: the longest one put into order
])
def test_the_order_of_the_items_changes_nothing(batch, hq, hkv, S, flags):
    gen = torch.Generator(device="cuda").manual_seed(S)
    rng = np.random.default_rng(S)
    d, v = (np.zeros((hq, S), np.uint8) for _ in range(2))
    for h in range(hq):
        if h % 5:  # (a head without patterns has no listed tiles)
            d[h, : S if h == 1 else 1 + rng.integers(0, 700)] = 1
            v[h, rng.integers(0, S, 12)] = 1
    mask = B.build_mask(mode=B.DAM_FROM_PATTERNS, H=hq, L=0, S=S, diag_in=torch.from_numpy(d).cuda(), vert_in=torch.from_numpy(v).cuda(),
                        flags=flags)
    q, k, v_ = (torch.randn((batch, h, S, 128), generator=gen, device="cuda", dtype=torch.bfloat16) for h in (hq, hkv, hkv))
    ws = B.prefill_workspace(B.attn_params(q, k, v_, torch.empty_like(q), 128, 128, gather_rows=mask.gather_rows), "cuda")
    got = []
    for room in (ws, ws[:-ORDER]):
        ws.fill_(0xFF)
        out = torch.full_like(q, 7.0)
        got.append(B.dam_sparse_attn_prefill(q, k, v_, mask, out=out, ws=room, want_lse=True))
    with pytest.raises(RuntimeError):
        B.dam_sparse_attn_prefill(q, k, v_, mask, ws=ws[:-ORDER - 256])
    torch.cuda.synchronize()
    (o1, l1), (o2, l2) = got
    assert torch.equal(o1, o2) and torch.equal(l1, l2)
    assert not bool((o1 == 7.0).all(-1).any())
