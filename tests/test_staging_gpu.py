"""Prefill tiles staged from memory to LDS: key counts around the edges of the
tiles (64 keys at D = 64, 32 at D = 128) and of the three-stage ring (one to
seven tiles), in every dtype and workgroup layout, against the fp64 oracle by
the suite's rules (T1 and T2 of helpers.py); rows past a sequence's length,
which the last tile's view ends before, hold NaN and must not show."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_18656_amd as fa
from paper_2608_18656_amd.inputs import DTYPES, make_qkv

from helpers import check_against, default_scale

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
def test_key_counts_around_tiles(D, dtype):
    BC = 4096 // D
    scale = default_scale(D)
    for n in range(1, 8):
        for Nk in (n * BC - 1, n * BC, n * BC + 1):
            for causal in (False, True):
                Nq = min(Nk, 40)
                if Nq == 1:
                    continue
                q, k, v = make_qkv(1, 8, 2, Nq, Nk, D, dtype, seed=100 * n + Nk)
                o_ref, l_ref = oracle.attention(q, k, v, causal, scale)
                qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
                for out in (torch.float32, None):
                    o, lse = fa.fwd(qd, kd, vd, causal=causal, scale=scale, out_dtype=out)
                    check_against(o, lse, o_ref, l_ref, DTYPES[dtype], out is not None, f"{Nk} {causal}")
                for slots in (1, 2, 8):
                    ox, lx = fa.fwd(qd, kd, vd, causal=causal, scale=scale, slots_per_workgroup=slots)
                    assert torch.equal(ox, o) and torch.equal(lx, lse), (Nk, causal, slots)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("page", [0, 64])
def test_rows_past_the_length_are_not_read(D, dtype, page):
    B, Hq, Hkv, Nq, Nk = 6, 8, 2, 5, 256
    lens = [256, 255, 129, 64, 31, 5]
    q, k, v = make_qkv(B, Hq, Hkv, Nq, Nk, D, dtype, seed=31)
    scale = default_scale(D)
    for b, n in enumerate(lens):
        k[b, n:] = float("nan")
        v[b, n:] = float("nan")
    sl = torch.tensor(lens, dtype=torch.int32).cuda()
    if page:
        table = torch.arange(B * Nk // page, dtype=torch.int32).view(B, -1).cuda()
        pool = [t.view(B * Nk // page, page, Hkv, D).cuda() for t in (k, v)]
        o, lse = fa.fwd_kvcache_paged(q.cuda(), *pool, table, sl, causal=True, scale=scale, out_dtype=torch.float32)
    else:
        o, lse = fa.fwd_kvcache(q.cuda(), k.cuda(), v.cuda(), sl, causal=True, scale=scale, out_dtype=torch.float32)
    for b, n in enumerate(lens):
        o_ref, l_ref = oracle.attention(q[b:b + 1], k[b:b + 1, :n], v[b:b + 1, :n], True, scale)
        check_against(o[b:b + 1], lse[b:b + 1], o_ref, l_ref, DTYPES[dtype], True, f"length {n}")


@pytest.mark.parametrize("B,Hq,Hkv,Nq", [(3, 7, 7, 70), (5, 9, 3, 33), (2, 12, 6, 65), (7, 5, 1, 34)])
def test_workgroup_numbering(B, Hq, Hkv, Nq):
    """Batches, heads and row blocks that divide nothing: each workgroup's
    place comes from its number by multiplication."""
    q, k, v = make_qkv(B, Hq, Hkv, Nq, Nq, 64, "f16", seed=B * 100 + Hq)
    scale = default_scale(64)
    o, lse = fa.fwd(q.cuda(), k.cuda(), v.cuda(), causal=True, scale=scale, out_dtype=torch.float32)
    o_ref, l_ref = oracle.attention(q, k, v, True, scale)
    check_against(o, lse, o_ref, l_ref, torch.float16, True)
    assert np.isfinite(o.cpu().numpy()).all()
