"""Lists of one row straight from the pattern flags: rows around the pieces of eight keys and the spans of 2048 keys that the
kernels work in, flag rows of odd length (so of every alignment), rows inside and below a true-mask block."""
import ctypes

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


def patterns_of(H, S, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    d, v = ((torch.rand((H, S), generator=gen, device="cuda") < 0.02).to(torch.uint8) for _ in range(2))
    for h in range(H):
        d[h, : 37 * (h % 9)] = 1
        v[h, S // 2:S // 2 + 11 * (h % 5)] = 1 + h % 255  # (any value but zero is a match)
    return d, v


def lists_of(d, v, row, G):
    """kept_ptr, kept_idx, kept_member of a row from the flags: runs of keys of two maps or more, then of each map alone."""
    bits = 1 << torch.arange(G, device="cuda")
    idx, mem, ptr = [], [], [0]
    for g in range(d.shape[0] // G):
        keep = (d[g * G:(g + 1) * G, :row + 1].flip(1) | v[g * G:(g + 1) * G, :row + 1]) != 0
        n = keep.sum(0)
        for run in ([n >= 2] if G > 1 else []) + [keep[x] & (n == 1) for x in range(G)]:
            at = run.nonzero().flatten()
            idx.append(at)
            mem.append((keep[:, at] * bits[:, None]).sum(0))
        ptr.append(sum(x.numel() for x in idx))
    return ptr, torch.cat(idx), torch.cat(mem)


# a workgroup per list: rows at the edges of 8, 16 and 32 keys per lane, of the flags and of what one launch takes (32768 keys, 64
# lists, 16384 keys of eight maps); built by the entry point, and with every total counted again instead of learned
@pytest.mark.parametrize("H,G,S,rows", [
    (3, 1, 8, (0, 3, 6, 7)), (16, 1, 4160, (4095, 4096, 4159)), (8, 4, 8200, (8190, 8191, 8192, 8199)), (6, 3, 16390, (16383, 16384, 16389)),
    (8, 4, 32800, (32759, 32767, 32768)), (64, 1, 20000, (19999,)), (65, 1, 300, (299,)), (16, 8, 16500, (16383, 16384)), (5, 1, 33, (7, 31, 32)),
])
def test_lists_in_one_launch(H, G, S, rows):
    d, v = patterns_of(H, S, S)
    for row in rows:
        m = B.build_mask(mode=B.DAM_FROM_PATTERNS, H=H, L=0, S=S, diag_in=d, vert_in=v, blocks=False, group=G if G > 1 else 0, rows=(row, row + 1))
        torch.cuda.synchronize()
        ptr, idx, mem = lists_of(d, v, row, G)
        n = ptr[-1]
        assert m.kept_ptr.tolist() == ptr and m.n_kept == n
        assert torch.equal(m.kept_idx[:n].long(), idx) and (G == 1 or torch.equal(m.kept_member[:n].long(), mem))
        p = B.MaskParams(B.DAM_FROM_PATTERNS, H, 0, S, 128, 128, row, row + 1, 0.5, 1e-8, 0.3, 0.8, float("nan"),
                         B.DAM_MASK_GROUP_LISTS if G > 1 else 0, 0, G if G > 1 else 0)
        again = {k: torch.full((n + 5,), 7, dtype=t, device="cuda") for k, t in (("idx", torch.int32), ("mem", torch.uint8))}
        kept_ptr, total = torch.full((H // G + 1,), -7, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda")
        o = B.MaskOut()
        o.kept_ptr, o.kept_idx, o.kept_total, o.kept_capacity = kept_ptr.data_ptr(), again["idx"].data_ptr(), total.data_ptr(), n - 1
        if G > 1:
            o.kept_member = again["mem"].data_ptr()
        ws = B.mask_workspace(p, "cuda")
        st = B.lib().dam_probe_row_lists(ctypes.byref(p), d.data_ptr(), v.data_ptr(), ctypes.byref(o), ws.data_ptr(), ws.numel(),
                                         torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        if H // G > 64 or row >= 32768 or (G > 4 and row >= 16384) or (S <= 64 and G == 1):
            assert st == -2  # DAM_ERR_UNSUPPORTED: the other way
            continue
        assert st == 0 and int(total) == n and kept_ptr.tolist() == [min(x, n - 1) for x in ptr]
        assert torch.equal(again["idx"][:n - 1].long(), idx[:n - 1]) and bool((again["idx"][n - 1:] == 7).all())
        assert G == 1 or torch.equal(again["mem"][:n - 1].long(), mem[:n - 1])


# the two launches: more lists than one launch takes, or flags off a multiple of eight bytes where a lane would read 128 of them.
# The piece at the row's end with one to eight keys, maps of fewer flags than a piece has
@pytest.mark.parametrize("H,G,S,rows", [
    (66, 1, 2061, range(2040, 2061)), (132, 2, 45, range(0, 45, 3)), (264, 4, 4099, range(4090, 4099)), (528, 8, 77, range(60, 77)),
    (66, 1, 5, range(5)), (132, 2, 8, range(8)), (8, 4, 20011, range(20000, 20011, 3)), (16, 8, 9003, (9000, 9002)),
])
def test_pieces_at_the_end_of_a_row(H, G, S, rows):
    d, v = patterns_of(H, S, S)
    for row in rows:
        m = B.build_mask(mode=B.DAM_FROM_PATTERNS, H=H, L=0, S=S, diag_in=d, vert_in=v, blocks=False, group=G if G > 1 else 0, rows=(row, row + 1))
        torch.cuda.synchronize()
        ptr, idx, mem = lists_of(d, v, row, G)
        n = ptr[-1]
        assert m.kept_ptr.tolist() == ptr and m.n_kept == n
        if n:
            assert torch.equal(m.kept_idx[:n].long(), idx) and (G == 1 or torch.equal(m.kept_member[:n].long(), mem))


# rows behind the flags' end: offsets and columns up to the capture's length only
@pytest.mark.parametrize("L", [5, 8, 9, 100, 2050])
@pytest.mark.parametrize("G", [1, 4])
def test_rows_past_the_flags(L, G):
    gen = torch.Generator(device="cuda").manual_seed(L)
    A = torch.rand((8, L, L), generator=gen, device="cuda").pow(6).tril()
    listed = 0
    for row in (*range(L, L + 18), 2 * L + 1, 4500):
        m = B.build_mask(mode=B.DAM_FROM_ATTN_MAP, H=8, L=L, S=4600, tau=0.5, mu=0.4, attn_sum=A, blocks=False, group=G if G > 1 else 0,
                         rows=(row, row + 1))
        torch.cuda.synchronize()
        d, v = (torch.nn.functional.pad(x, (0, row + 1 - L)) for x in (m.diag_flag, m.vert_flag))
        ptr, idx, mem = lists_of(d, v, row, G)
        n = ptr[-1]
        listed += n
        assert m.kept_ptr.tolist() == ptr and m.n_kept == n
        if n:
            assert torch.equal(m.kept_idx[:n].long(), idx) and (G == 1 or torch.equal(m.kept_member[:n].long(), mem))
    assert listed > 0
