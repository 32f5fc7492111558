"""Chunks of prompts against long caches, D = 64, on grids where the default is
eight slots per workgroup (32 x 32/8 heads, 128 rows, 2048 keys: two full rounds)
and just past them (a third round that would be nearly empty, 2047 keys): bit for
bit the four-slot results."""
import pytest
import torch

import paper_2608_18656_amd as fa
from paper_2608_18656_amd.inputs import make_qkv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Nk,dtype", [(32, 2048, "bf16"), (32, 2047, "f16"), (33, 2048, "f16")])
def test_chunks(B, Nk, dtype):
    q, k, v = (t.cuda() for t in make_qkv(B, 32, 8, 128, Nk, 64, dtype, seed=Nk + B))
    for causal in (True, False):
        o, lse = fa.fwd(q, k, v, causal=causal, out_dtype=torch.float32)
        o4, l4 = fa.fwd(q, k, v, causal=causal, out_dtype=torch.float32, slots_per_workgroup=4)
        assert torch.equal(o, o4) and torch.equal(lse, l4)
        full = torch.full((B,), Nk, dtype=torch.int32, device="cuda")
        oc, lc = fa.fwd_kvcache(q, k, v, full, causal=causal, out_dtype=torch.float32)
        assert torch.equal(oc, o4) and torch.equal(lc, l4)
    lens = full - torch.arange(B, dtype=torch.int32, device="cuda") * (Nk - 100) // (B - 1)
    o, lse = fa.fwd_kvcache(q, k, v, lens, causal=True, out_dtype=torch.float32)
    for b in (0, 1, B // 2, B - 1):   # one sequence alone takes four slots
        ob, lb = fa.fwd_kvcache(q[b:b + 1], k[b:b + 1], v[b:b + 1], lens[b:b + 1], causal=True, out_dtype=torch.float32)
        assert torch.equal(o[b:b + 1], ob) and torch.equal(lse[b:b + 1], lb), b
