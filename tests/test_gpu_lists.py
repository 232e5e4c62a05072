"""Lists of one row straight from the pattern flags: rows around the pieces of eight keys and the spans of 2048 keys that the
kernels work in, flag rows of odd length (so of every alignment), rows inside and below a true-mask block."""
import numpy as np
import pytest
import torch

from paper_2506_11104_amd import binding as B
from test_gpu_decode import group_lists_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,H,S,L,rows", [
    (1, 3, 4101, 0, (0, 6, 7, 8, 2047, 2048, 2049, 4095, 4096, 4100)), (4, 8, 6151, 0, (2046, 2055, 6150)),
    (8, 8, 2049, 0, (2048,)), (2, 6, 333, 203, (195, 199, 202, 203, 210, 211, 332)),
])
def test_rows_around_pieces_and_spans(G, H, S, L, rows):
    rng = np.random.default_rng(S + G)
    dflag, vflag = ((rng.random((H, S)) < 0.03).astype(np.uint8) for _ in range(2))
    for h in range(H):
        dflag[h, : 5 * h] = 1
        vflag[h, -3:] = 1
    tm = np.tril(rng.random((H, L, L)) < 0.3).astype(np.uint8) if L else None
    for row in rows:
        group_lists_case(H, G, S, row, dflag, vflag, **({"L": L, "true_mask": tm} if L else {}))


@pytest.mark.parametrize("H,G,spans", [(64, 1, 96), (64, 1, 97), (48, 8, 227), (48, 8, 228)])
def test_lists_on_both_sides_of_the_scan(H, G, spans):
    """12288 counts are the most whose sum every workgroup forms itself: lists of as many, and of one span of 2048 keys more."""
    S = 2048 * spans - 5
    gen = torch.Generator(device="cuda").manual_seed(spans)
    d, v = ((torch.rand((H, S), generator=gen, device="cuda") < 0.002).to(torch.uint8) for _ in range(2))
    m = B.build_mask(mode=B.DAM_FROM_PATTERNS, H=H, L=0, S=S, diag_in=d, vert_in=v, blocks=False, group=G, rows=(S - 1, S))
    torch.cuda.synchronize()
    idx, mem, ptr = [], [], [0]
    bits = 1 << torch.arange(G, device="cuda")
    for g in range(H // G):
        keep = (d[g * G:(g + 1) * G].flip(1) | v[g * G:(g + 1) * G]) != 0
        n = keep.sum(0)
        for run in [n >= 2] + [keep[x] & (n == 1) for x in range(G)]:
            at = run.nonzero().flatten()
            idx.append(at)
            mem.append((keep[:, at] * bits[:, None]).sum(0))
        ptr.append(sum(x.numel() for x in idx))
    assert m.n_kept == ptr[-1] and m.kept_ptr.tolist() == ptr
    assert torch.equal(m.kept_idx[:ptr[-1]].long(), torch.cat(idx)) and torch.equal(m.kept_member[:ptr[-1]].long(), torch.cat(mem))
