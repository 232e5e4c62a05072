"""Lists split over several workgroups, the last of which merges them (no launch of its own, flags in a workspace that is
never cleared): against the oracle from a workspace full of ones, and replayed from a HIP graph with another call on the
same workspace in between."""
import numpy as np
import pytest
import torch

import oracle
from dam_testlib import dev
from paper_2506_11104_amd import binding as B
from paper_2506_11104_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-4, "bf16": 2e-2}


def problem(dtype, d, Bn, Hkv, G, longest, grouped, seed):
    rng = np.random.default_rng(seed)
    Hq, T = Hkv * G, longest + 50
    q, Kc, Vc = (wl.to_storage(rng.standard_normal(s).astype(np.float32), dtype) for s in ((Bn, Hq, d), (Bn, Hkv, T, d), (Bn, Hkv, T, d)))
    lens = [longest if h % 3 == 0 else (0 if h % 3 == 1 else longest // 2 + 1) for h in range(Hq)]
    lists = [np.sort(rng.choice(T, n, replace=False)).astype(np.int32) for n in lens]
    kv_of = np.array([b * Hkv + h // G for b in range(Bn) for h in range(Hq)], np.int32)
    ptr = np.concatenate([[0], np.cumsum(lens * Bn)]).astype(np.int64)
    O, LSE = oracle.attend_lists(q.reshape(-1, d), Kc.reshape(-1, T, d), Vc.reshape(-1, T, d), kv_of, ptr, np.concatenate(lists * Bn))
    if grouped:
        gp, gi, gm = oracle.group_lists(lists, G)
    else:
        gp, gi, gm = np.concatenate([[0], np.cumsum(lens)]), np.concatenate(lists), None
    t = lambda a, k: torch.from_numpy(np.ascontiguousarray(a.astype(k))).cuda()
    args = [dev(q, dtype), dev(Kc, dtype), dev(Vc, dtype), t(gp, np.int32), t(gi, np.int32)] + ([t(gm, np.uint8)] if grouped else [])
    most = int(np.diff(gp).max())
    out, lse = torch.empty_like(args[0]), torch.empty((Bn, Hq), device="cuda")
    p = B.decode_params(args[0], args[1], out, shared_lists=True)
    need = (B.decode_grouped_workspace if grouped else B.decode_workspace)(p, most, "cuda").numel()

    def run(ws):
        (B.dam_sparse_attn_decode_grouped if grouped else B.dam_sparse_attn_decode)(*args, most, out=out, lse=lse, ws=ws, shared_lists=True)

    def check():
        torch.cuda.synchronize()
        assert np.abs(out.float().cpu().numpy().reshape(-1, d) - O).max() <= TOL[dtype]
        got = lse.cpu().numpy().reshape(-1)
        assert np.array_equal(np.isneginf(got), np.isneginf(LSE)) and np.abs(np.where(np.isneginf(LSE), 0, got - LSE)).max() <= TOL[dtype]
        out.fill_(7.0)
        lse.fill_(7.0)
    return run, check, need


@pytest.mark.parametrize("dtype,d,Bn,Hkv,G,longest,grouped", [
    ("bf16", 128, 1, 1, 8, 3000, True),      # 16 groups of four waves
    ("bf16", 128, 2, 3, 3, 640, True),       # a column count that does not divide the workgroup
    ("bf16", 128, 3, 2, 1, 129, True), ("bf16", 128, 5, 17, 2, 700, True), ("bf16", 128, 1, 2, 4, 130, True),
    ("f32", 64, 1, 2, 2, 17000, False),      # 64 splits
    ("bf16", 64, 3, 1, 4, 520, False), ("bf16", 128, 1, 4, 2, 1100, False),
    ("f32", 128, 1, 2, 8, 1500, True), ("bf16", 64, 1, 1, 3, 900, True),
])
def test_split_lists(dtype, d, Bn, Hkv, G, longest, grouped):
    run, check, need = problem(dtype, d, Bn, Hkv, G, longest, grouped, 11 + longest)
    other, check_other, need_other = problem(dtype, d, 1, Hkv, G, longest // 2 + 200, grouped, 12)
    ws = torch.full((max(need, need_other),), 0xFF, dtype=torch.uint8, device="cuda")
    run(ws)
    check()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run(ws)
    for k in range(4):
        g.replay()
        check()
        if k % 2:
            other(ws)
            check_other()


@pytest.mark.parametrize("Bn,n", [(1, 20), (1, 100), (1, 300), (1, 3000), (16, 600), (64, 5000)])
def test_nan_logits_come_out_as_nan_however_the_list_is_split(Bn, n):
    """One wave, several, several workgroups. Head 1's query is NaN and head 2 keeps no key, while every key of KV head 1's
    list is NaN: the outputs are NaN for head 1 and for KV head 1's heads with keys, zero for its head without, and ordinary
    for the others."""
    Hkv, G, d, T = 2, 4, 128, n + 40
    rng = np.random.default_rng(n)
    q, Kc, Vc = (wl.to_storage(rng.standard_normal(s).astype(np.float32), "bf16") for s in ((Bn, 8, d), (Bn, Hkv, T, d), (Bn, Hkv, T, d)))
    lists = [np.sort(rng.choice(T, n, replace=False)).astype(np.int32) for _ in range(8)]
    lists[2] = lists[6] = np.zeros(0, np.int32)
    kv_of = np.array([b * Hkv + h // G for b in range(Bn) for h in range(8)], np.int32)
    ptr = np.concatenate([[0], np.cumsum([x.size for x in lists] * Bn)]).astype(np.int64)
    O, _ = oracle.attend_lists(q.reshape(-1, d), Kc.reshape(-1, T, d), Vc.reshape(-1, T, d), kv_of, ptr, np.concatenate(lists * Bn))
    gp, gi, gm = oracle.group_lists(lists, G)
    q[:, 1] = np.nan
    Kc[:, 1] = np.nan
    t = lambda a, k: torch.from_numpy(np.ascontiguousarray(a.astype(k))).cuda()
    out, lse = B.dam_sparse_attn_decode_grouped(dev(q, "bf16"), dev(Kc, "bf16"), dev(Vc, "bf16"), t(gp, np.int32), t(gi, np.int32),
                                                t(gm, np.uint8), int(np.diff(gp).max()), want_lse=True, shared_lists=True)
    torch.cuda.synchronize()
    out, O = out.float().cpu().numpy(), O.reshape(Bn, 8, d)
    assert np.isnan(out[:, [1, 4, 5, 7]]).all()
    assert (out[:, [2, 6]] == 0).all() and bool(torch.isneginf(lse[:, [2, 6]]).all())
    assert np.abs(out[:, [0, 3]] - O[:, [0, 3]]).max() <= TOL["bf16"]
