"""The items of the bf16 prefill that are computed again with a running reference, where a workgroup takes several items: a
launch has at most two workgroups per CU (512), and what it takes beyond its first item it draws from the queues."""
import numpy as np
import pytest
import torch

import oracle
from dam_testlib import dev
from paper_2506_11104_amd import binding as B
from paper_2506_11104_amd import workloads as wl
from test_gpu_prefill import gpu_mask_from_art

pytestmark = pytest.mark.gpu
TOL = 2e-2


def qkv(seed, H, S):
    rng = np.random.default_rng(seed)
    return [wl.to_storage(rng.standard_normal((H, S, 128)).astype(np.float32), "bf16") for _ in range(3)]


def patterns(H, S):
    d, v = (np.zeros((H, S), np.uint8) for _ in range(2))
    for h in range(H):
        d[h, : 20 + 9 * h] = 1
        v[h, 3 + h :: 700] = 1
    return oracle.from_patterns(d, v)


def against_oracle(got, lse, Q, K, V, art, scale):
    O, LSE = oracle.attend_prefill(Q, K, V, art, scale=scale or None)
    assert np.abs(got.float().cpu().numpy() - O).max() <= TOL
    # a logit is a sum of 128 products: its fp32 error, and so that of the log-sum-exp, grows with it
    assert np.abs(lse.cpu().numpy() - LSE).max() <= TOL * max(1.0, np.abs(LSE).max() / 500)


@pytest.mark.parametrize("polluted_first,flags", [(False, 0), (True, B.DAM_ATTN_RUNNING_REFERENCE)])
def test_a_sequence_with_nan_values_leaves_its_neighbour_alone(polluted_first, flags):
    """Two sequences of 16 heads x 4096 tokens, 1024 items: a workgroup takes items of the first, then of the second. One has
    NaN in every V row; the other's items are done with the running reference, behind the first kind (logits beyond the
    plain exponential, or the flag) and must not meet those rows."""
    H, S = 16, 4096
    Q, K, V = qkv(5, H, S)
    art = patterns(H, S)
    mask = gpu_mask_from_art(art, S, 128, 128)
    q, k, v = (torch.stack([dev(x, "bf16")] * 2) for x in (Q, K, V))
    bad = 0 if polluted_first else 1
    v[bad] = float("nan")
    q[1 - bad] *= 64.0
    out, lse = B.dam_sparse_attn_prefill(q, k, v, mask, want_lse=True, flags=flags)
    torch.cuda.synchronize()
    assert bool(torch.isnan(out[bad]).all())
    against_oracle(out[1 - bad], lse[1 - bad], Q * 64.0, K, V, art, 0.0)


@pytest.mark.parametrize("Hq,Hkv,S,odd_only,flags", [
    (16, 16, 4096, False, 0), (16, 4, 4001, False, B.DAM_MASK_GATHER_COLUMNS), (16, 8, 4096, True, B.DAM_MASK_GATHER_COLUMNS),
    (6, 3, 6001, False, 0), (6, 3, 6016, True, 0),     # six pairs: round robin over the queues
])
def test_workgroups_redo_several_items(Hq, Hkv, S, odd_only, flags):
    """564 to 1024 items, all of them (or those of every other head) beyond the plain exponential: the lists of items to
    redo have several entries, of first items and of drawn ones, in both layouts, whole and ragged."""
    Q, K, V = qkv(7 + S, Hq, S)
    K, V = K[:Hkv], V[:Hkv]
    Q[1 if odd_only else 0 :: 2 if odd_only else 1] *= 64.0
    art = patterns(Hq, S)
    mask = gpu_mask_from_art(art, S, 128, 128, flags=flags)
    q, k, v = (torch.stack([dev(x, "bf16")] * 2) for x in (Q, K, V))
    # Every sum and rounding scales with V by a power of two, but for outputs below bf16's normal range, 2^-126. (Negated
    # values do not: the matrix instruction's sums round 18 of 8 388 608 outputs another way, redone or not.)
    v[1] *= 2
    out, lse = B.dam_sparse_attn_prefill(q, k, v, mask, want_lse=True)
    torch.cuda.synchronize()
    against_oracle(out[0], lse[0], Q, K, V, art, 0.0)
    assert float((out[1].float() - 2 * out[0].float()).abs().max()) <= 2.0 ** -126 and torch.equal(lse[1], lse[0])


@pytest.mark.parametrize("B_,Hq,Hkv,S,flags", [
    (1, 8, 2, 2048, 0), (1, 4, 4, 1000, B.DAM_MASK_GATHER_COLUMNS), (2, 16, 8, 2048, B.DAM_MASK_GATHER_COLUMNS), (1, 6, 3, 257, 0),
])
def test_workgroups_redo_their_only_item(B_, Hq, Hkv, S, flags):
    """18 to 512 items, one to a workgroup, all of them beyond the plain exponential: every list has exactly one entry, so that it
    is empty again as soon as wave 0 has taken it, and every wave's rows have to be those of the second variant all the same."""
    Q, K, V = qkv(11 + S, Hq, S)
    K, V = K[:Hkv], V[:Hkv]
    Q *= 64.0
    art = patterns(Hq, S)
    mask = gpu_mask_from_art(art, S, 128, 128, flags=flags)
    q, k, v = (torch.stack([dev(x, "bf16")] * B_) for x in (Q, K, V))
    out, lse = B.dam_sparse_attn_prefill(q, k, v, mask, want_lse=True)
    torch.cuda.synchronize()
    for b in range(B_):
        against_oracle(out[b], lse[b], Q, K, V, art, 0.0)
