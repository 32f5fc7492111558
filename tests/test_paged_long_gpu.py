"""Prefill against long block tables: a wave holds 64 entries of its
sequence's row and the next 64, so rows of just under, at and past 64, 128 and
192 pages (bitwise as the contiguous cache)."""
import pytest
import torch

import paper_2608_18656_amd as fa
from paper_2608_18656_amd.inputs import make_qkv

from test_paged_gpu import _paginate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,dt,Nq,causal", [(64, "f16", 40, True), (64, "bf16", 130, True), (128, "f16", 33, False),
                                            (128, "bf16", 70, True)])
@pytest.mark.parametrize("pages", [63, 64, 65, 129, 193])
def test_many_pages(pages, D, dt, Nq, causal):
    B, Hq, Hkv, page = 3, 4, 2, 64
    Nk = pages * page
    q, k, v = make_qkv(B, Hq, Hkv, Nq, Nk, D, dt, seed=pages + D)
    kp, vp, table = (t.cuda() for t in _paginate(k, v, page, pages))
    sl = torch.tensor([Nk, Nk - page + 1, max(Nk // 2, Nq)], dtype=torch.int32).cuda()
    q, k, v = q.cuda(), k.cuda(), v.cuda()
    o, lse = fa.fwd_kvcache_paged(q, kp, vp, table, sl, causal=causal, out_dtype=torch.float32)
    oc, lc = fa.fwd_kvcache(q, k, v, sl, causal=causal, out_dtype=torch.float32)
    assert torch.isfinite(o).all()
    assert torch.equal(o, oc) and torch.equal(lse, lc)
