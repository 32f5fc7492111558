"""Workgroups of a batch with uneven lengths are started by length (2 to 64
sequences, grids past one workgroup per CU); the order must not show in the
results.  Prefill: every sequence equals, bit for bit, a call of its own.
Decode (whose split count depends on the batch): the oracle, and bitwise the
same batch in another order."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_18656_amd as fa
from paper_2608_18656_amd.inputs import DTYPES, make_qkv

from helpers import check_against, default_scale

pytestmark = pytest.mark.gpu


def _lengths(B, Nk, least, seed):
    """Uneven: the full length, an equal pair, the least, 0 where allowed, and between."""
    rng = np.random.default_rng(seed)
    n = rng.integers(max(least, Nk // 6), Nk, size=B)
    n[rng.permutation(B)[:2]] = Nk // 2
    n[int(rng.integers(B))] = Nk
    n[-1] = least
    return n.tolist()


# B, Hq, Hkv, Nq, Nk, D, causal, dtype: 2 to 64 sequences in one or several
# rounds of workgroups, 65 (not ordered), non-causal, row blocks of 32 to 128
@pytest.mark.parametrize("case", [(2, 64, 16, 300, 500, 64, True, "bf16"), (5, 16, 16, 500, 640, 64, True, "f16"),
                                  (7, 64, 8, 200, 333, 128, True, "bf16"), (64, 4, 2, 300, 310, 64, True, "bf16"),
                                  (9, 32, 8, 150, 400, 128, False, "f16"), (65, 4, 2, 300, 310, 64, True, "f16")],
                         ids=lambda c: "x".join(map(str, c)))
def test_prefill_sequences_equal_their_own_calls(case):
    B, Hq, Hkv, Nq, Nk, D, causal, dt = case
    q, k, v = (t.cuda() for t in make_qkv(B, Hq, Hkv, Nq, Nk, D, dt, seed=70 + B))
    for lens in (_lengths(B, Nk, 17, B), [Nk - b % 2 for b in range(B)]):   # uneven; about equal
        sl = torch.tensor(lens, dtype=torch.int32).cuda()
        o, lse = fa.fwd_kvcache(q, k, v, sl, causal=causal, out_dtype=torch.float32)
        for b in range(B):
            ob, lb = fa.fwd_kvcache(q[b:b + 1], k[b:b + 1], v[b:b + 1], sl[b:b + 1], causal=causal,
                                    out_dtype=torch.float32)
            assert torch.equal(o[b:b + 1], ob) and torch.equal(lse[b:b + 1], lb), (b, lens[b])


@pytest.mark.parametrize("case", [(40, 16, 16, 640, 64, "f16", 64), (64, 32, 8, 520, 128, "bf16", 0),
                                  (33, 8, 8, 1088, 64, "bf16", 0), (65, 8, 8, 600, 128, "f16", 0)],
                         ids=lambda c: "x".join(map(str, c)))
def test_decode(case):
    B, Hq, Hkv, Nk, D, dt, page = case
    q, k, v = make_qkv(B, Hq, Hkv, 1, Nk, D, dt, seed=90 + B)
    lens = _lengths(B, Nk, 0, B)
    scale = default_scale(D)

    def call(order):
        qd, kd, vd = (t[order].contiguous().cuda() for t in (q, k, v))
        sl = torch.tensor([lens[b] for b in order], dtype=torch.int32).cuda()
        if not page:
            return fa.fwd_kvcache(qd, kd, vd, sl, causal=True, scale=scale, out_dtype=torch.float32)
        pages = [t.reshape(B * Nk // page, page, Hkv, D) for t in (kd, vd)]
        table = torch.arange(B * Nk // page, dtype=torch.int32).view(B, -1).cuda()
        return fa.fwd_kvcache_paged(qd, *pages, table, sl, causal=True, scale=scale, out_dtype=torch.float32)

    o, lse = call(list(range(B)))
    other = np.random.default_rng(1).permutation(B).tolist()
    op, lp = call(other)
    assert torch.equal(op, o[other]) and torch.equal(lp, lse[other])
    for b, n in enumerate(lens):
        if n == 0:
            assert torch.all(o[b] == 0) and torch.all(torch.isneginf(lse[b]))
            continue
        o_ref, l_ref = oracle.attention(q[b:b + 1], k[b:b + 1, :n].contiguous(), v[b:b + 1, :n].contiguous(), True, scale)
        check_against(o[b:b + 1], lse[b:b + 1], o_ref, l_ref, DTYPES[dt], True, f"{case} b={b} n={n}")
