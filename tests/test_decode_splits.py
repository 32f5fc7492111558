"""Decode split counts: the default's bounds (CPU), and on the GPU the single
split that writes its result directly and the splits of sequences of
different lengths, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_18656_amd as fa
from paper_2608_18656_amd.inputs import DTYPES, make_qkv

from helpers import check_against, default_scale


def _splits(B, Hq, Hkv, Nk, D):
    return fa.workspace_bytes(B, Hq, Hkv, 1, Nk, D, "f16") // (B * Hq * (D + 2) * 4)


def test_default_split_bounds():
    for D in (64, 128):
        for B in (1, 3, 16, 41, 64, 300, 5000):
            for Hq, Hkv in ((32, 8), (16, 1), (16, 16), (48, 2)):
                units = B * Hkv * -(-(Hq // Hkv) // 16)
                for Nk in (1, 31, 256, 257, 512, 1537, 4096, 8839, 131072, 2**31 - 1):
                    S = _splits(B, Hq, Hkv, Nk, D)
                    assert 1 <= S <= min(256, -(-Nk // 256)), (B, Hq, Hkv, Nk, D, S)
                    # splitting stops at eight rounds of one workgroup a CU
                    assert S == 1 or units * S <= 8 * 256, (B, Hq, Hkv, Nk, D, S)


@pytest.mark.gpu
@pytest.mark.parametrize("D,dtype", [(64, "f16"), (64, "bf16"), (128, "f16"), (128, "bf16")])
@pytest.mark.parametrize("Nk", [1, 31, 32, 33, 255, 257, 300])
def test_single_split_writes_the_result(D, dtype, Nk):
    B, Hq, Hkv = 2, 34, 2   # two query groups of 16 and 1 heads
    assert _splits(B, Hq, Hkv, Nk, D) == 1
    q, k, v = make_qkv(B, Hq, Hkv, 1, Nk, D, dtype, seed=Nk + D)
    scale = default_scale(D)
    o_ref, l_ref = oracle.attention(q, k, v, False, scale)
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    for out in (torch.float32, None):
        o, lse = fa.fwd(qd, kd, vd, scale=scale, out_dtype=out)
        check_against(o, lse, o_ref, l_ref, DTYPES[dtype], out is not None)
    o2, none = fa.fwd(qd, kd, vd, scale=scale, return_lse=False)
    assert none is None and torch.equal(o2, o)


@pytest.mark.gpu
@pytest.mark.parametrize("D,dtype,page", [(64, "bf16", 0), (64, "f16", 64), (128, "bf16", 128), (128, "f16", 0)])
@pytest.mark.parametrize("Nk", [384, 2048])
def test_lengths_spread_over_the_splits(D, dtype, page, Nk):
    lens = [Nk, Nk - 1, Nk // 2 + 1, 257, 33, 32, 1, 0]
    B, Hq, Hkv = len(lens), 6, 2
    q, k, v = make_qkv(B, Hq, Hkv, 1, Nk, D, dtype, seed=Nk + D)
    for b, n in enumerate(lens):
        k[b, n:] = float("nan")
        v[b, n:] = float("nan")
    scale = default_scale(D)
    sl = torch.tensor(lens, dtype=torch.int32).cuda()
    kd, vd = k.cuda(), v.cuda()
    o, lse = fa.fwd_kvcache(q.cuda(), kd, vd, sl, scale=scale, out_dtype=torch.float32)
    for b, n in enumerate(lens):
        if n == 0:
            assert torch.all(o[b] == 0) and torch.all(lse[b] == -float("inf"))
            continue
        o_ref, l_ref = oracle.attention(q[b:b + 1], k[b:b + 1, :n], v[b:b + 1, :n], False, scale)
        check_against(o[b:b + 1], lse[b:b + 1], o_ref, l_ref, DTYPES[dtype], True, f"length {n}")
    if page:
        order = torch.from_numpy(np.random.default_rng(1).permutation(B * Nk // page).astype(np.int32)).cuda()
        pools = []
        for t in (kd, vd):
            pool = torch.empty((B * Nk // page, page, Hkv, D), dtype=t.dtype, device="cuda")
            pool[order.long()] = t.view(-1, page, Hkv, D)
            pools.append(pool)
        op, lp = fa.fwd_kvcache_paged(q.cuda(), *pools, order.view(B, -1), sl, scale=scale, out_dtype=torch.float32)
        assert torch.equal(op, o) and torch.equal(lp, lse)


@pytest.mark.gpu
@pytest.mark.parametrize("D,dtype", [(64, "bf16"), (64, "f16"), (128, "bf16"), (128, "f16")])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_scores_that_are_no_numbers(D, dtype, bad):
    """One split writes its own result: the same as the merge of several, 0 and -inf."""
    q, k, v = (t.cuda() for t in make_qkv(2, 6, 2, 1, 600, D, dtype, seed=D))
    q[0, 0, 1, 0], q[0, 0, 4, 0] = abs(q[0, 0, 1, 0]) + 1, abs(q[0, 0, 4, 0]) + 1
    k[0, 100, :, 0] = bad
    res = [fa.fwd(q, k, v, num_splits=S, scale=default_scale(D)) for S in (1, 3)]
    for o, lse in res:
        for h in (1, 4):
            assert torch.all(o[0, 0, h] == 0) and lse[0, h, 0] == -float("inf")
    assert not res[0][0].isnan().any() and torch.equal(res[0][1].isinf(), res[1][1].isinf())
    assert torch.equal(res[0][0] == 0, res[1][0] == 0)
