"""Captures whose row tiles are shared by up to four workgroups (stages of 64 keys, an even number per part), and the summed
form around its tiles of 32 rows and 256 keys, with row lengths that are whole 128-byte lines and that are not."""
import numpy as np
import pytest
import torch

import oracle
from dam_testlib import dev
from paper_2506_11104_amd import binding as B
from paper_2506_11104_amd import workloads as wl
from test_gpu_capture import ATOL, RTOL, fused_against_oracle, seq_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,L,Hq,Hkv", [(255, 256, 2, 1), (257, 288, 8, 8), (385, 385, 3, 3), (513, 515, 2, 2), (600, 640, 16, 8),
                                        (1025, 1026, 2, 1)])
def test_parts_and_tiles(n, L, Hq, Hkv):
    Q, K = seq_pair(700 + n, Hq, Hkv, n, 128, "bf16", std=1.2)
    A, C = oracle.capture(Q, K, L)
    a_dev, c_dev = (torch.zeros((Hq, L, L), dtype=torch.float32, device="cuda") for _ in range(2))
    ws = torch.full((B.capture_workspace(B.capture_params(dev(Q, "bf16"), dev(K, "bf16"), L), "cuda").numel(),), 0xFF,
                    dtype=torch.uint8, device="cuda")
    B.dam_capture_accumulate(dev(Q, "bf16"), dev(K, "bf16"), a_dev, c_dev, ws=ws)
    torch.cuda.synchronize()
    assert np.array_equal(c_dev.cpu().numpy(), C)
    err = np.abs(a_dev.cpu().numpy() - A)
    assert (err <= ATOL + RTOL * A).all(), err.max()
    w = wl.scaled(wl.WORKLOADS["c2"], hq=Hq, hkv=Hkv, seq=n, pcl=n)
    fused_against_oracle(Q, K, w, n, 128, 128, 0.05, 0.8, "bf16")


def test_sequences_of_several_lengths_in_one_workspace():
    """A workspace sized for the longest sequence takes shorter ones, which are cut into more parts. It ends in bytes that
    must stay as they are."""
    Hq, Hkv, L, lens = 32, 8, 2048, (2048, 300, 1000, 1)
    q, k = (dev(x, "bf16") for x in seq_pair(31, Hq, Hkv, L, 128, "bf16", std=1.2))
    need = B.capture_workspace(B.capture_params(q, k, L), "cuda").numel()
    ws = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    got, want = (torch.zeros((Hq, L, L), dtype=torch.float32, device="cuda") for _ in range(2))
    for n in lens:
        B.dam_capture_accumulate(q[:, :n], k[:, :n], got, None, ws=ws[:need])
        s = (q[:, :n].float().reshape(Hkv, -1, 128) @ k[:, :n].float().transpose(1, 2).contiguous()).reshape(Hq, n, n) / 128 ** 0.5
        want[:, :n, :n] += s.masked_fill(torch.ones((n, n), dtype=torch.bool, device="cuda").triu(1), float("-inf")).softmax(-1)
    torch.cuda.synchronize()
    assert bool(((got - want).abs() <= len(lens) * ATOL + RTOL * want).all())
    assert bool((ws[need:] == 0x5A).all())


def test_rows_in_several_parts_are_as_exact_as_rows_in_one():
    """The same heads captured alone (four parts per row tile) and among 80 (one): the error against 64 bits may not differ.
    Logits to about 40, where a log-sum-exp rounded to fp32 is off by up to 2^-19 and each further rounding of that
    size adds to the error of every probability (one per part made it 14 % larger here). The 2-norms of the
    two runs of 1.6 million roundings agree to well under 1 %; 2 % are allowed."""
    n, copies = 900, 20
    q, k = (dev(x, "bf16") for x in seq_pair(41, 4, 1, n, 128, "bf16"))
    q *= 5
    A1, A20 = torch.zeros((4, n, n), device="cuda"), torch.zeros((4 * copies, n, n), device="cuda")
    B.dam_capture_accumulate(q, k, A1)
    B.dam_capture_accumulate(q.repeat(copies, 1, 1), k.repeat(copies, 1, 1), A20)
    errors = []
    for A in (A1, A20[:4]):
        d2 = 0.0
        for h in range(4):
            s = (q[h].double() @ k[0].double().t()) / 128 ** 0.5
            p = s.masked_fill(torch.ones((n, n), dtype=torch.bool, device="cuda").triu(1), float("-inf")).softmax(-1)
            d2 += float((A[h].double() - p).pow(2).sum())
        errors.append(d2 ** 0.5)
    assert errors[0] <= 1.02 * errors[1], errors


@pytest.mark.parametrize("copies,first,last", [(1, 256, 512), (1, 0, 900), (1, 256, 900), (40, 0, 900), (40, 256, 512)])
def test_a_part_without_a_number_is_not_left_out(copies, first, last):
    """Keys [first, last) are NaN, whole parts of the rows that hold them: every probability of such a row is NaN, in one
    part (80 heads) and in several (2), and the rows above are those of a softmax over their own keys."""
    n = 900
    Q, K = seq_pair(43, 2, 1, n, 128, "bf16", std=1.2)
    A, _ = oracle.capture(Q, K, n, want_cnt=False)
    K[:, first:last] = np.nan
    a_dev = torch.zeros((2 * copies, n, n), dtype=torch.float32, device="cuda")
    B.dam_capture_accumulate(dev(Q, "bf16").repeat(copies, 1, 1), dev(K, "bf16").repeat(copies, 1, 1), a_dev, None)
    torch.cuda.synchronize()
    lower = np.tril(np.ones((n, n), bool))
    for got in a_dev[[0, 2 * copies - 1]].cpu().numpy():
        assert np.array_equal(np.isnan(got), lower & (np.arange(n) >= first)[:, None])
    got = a_dev[0, :first].cpu().numpy()
    assert (np.abs(got - A[0, :first]) <= ATOL + RTOL * A[0, :first]).all()


# 32 keys per wave up to 6144 workgroups of 64 keys, 64 beyond: the same four heads alone and among enough others, around the
# spans of 128 and 256 keys, rows of whole lines and not
@pytest.mark.parametrize("n,L", [(127, 128), (129, 130), (255, 256), (257, 288), (385, 385), (513, 515), (900, 900)])
def test_narrow_and_wide_tiles_of_the_sum(n, L):
    R = (n + 255) // 256
    copies = 6144 // (4 * 4 * R * (R + 1)) + 1
    q, k = (dev(x, "bf16") for x in seq_pair(47 + n, 4, 2, n, 128, "bf16", std=1.2))
    s = (q.double().reshape(2, 2 * n, 128) @ k.double().transpose(1, 2).contiguous()).reshape(4, n, n) / 128 ** 0.5
    want = s.masked_fill(torch.ones((n, n), dtype=torch.bool, device="cuda").triu(1), float("-inf")).softmax(-1)
    for c in (1, copies):
        A, C = (torch.full((4 * c, L, L), 0.25, device="cuda") for _ in range(2))
        B.dam_capture_accumulate(q.repeat(c, 1, 1), k.repeat(c, 1, 1), A, C)
        torch.cuda.synchronize()
        lower = torch.ones((L, L), dtype=torch.bool, device="cuda").tril_()
        lower[n:] = False
        assert bool((C == torch.where(lower, 1.25, 0.25)).all())
        assert bool((A[:, ~lower] == 0.25).all())
        got = A[[*range(4), *range(4 * c - 4, 4 * c)], :n, :n].double() - 0.25
        # (a quarter takes the probability's last bits: half an ulp of 0.5 and of 1)
        assert bool(((got - want.repeat(2, 1, 1)).abs().tril() <= 2.0 ** -24 + ATOL + RTOL * want.repeat(2, 1, 1)).all())
