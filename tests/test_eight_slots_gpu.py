"""D = 64 calls on both sides of the lines between four and eight slots per
workgroup: bit for bit the same results.  Chunks of prompts against long caches
(32 x 32/8 heads, 128 rows, 2048 keys: two full rounds of eight), with lengths
and without; short and long calls; a K/V larger than the memory side's cache."""
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


@pytest.mark.parametrize("shape", [
    (49, 32, 8, 57, 57, False, "f16"),       # two rounds of short calls: four slots
    (3, 32, 8, 712, 712, False, "bf16"),     # one round: eight from here on
    (3, 32, 8, 711, 711, False, "bf16"),
    (46, 16, 16, 136, 1800, False, "bf16"),  # K/V of 339 MB, read half as often by eight
    (46, 16, 16, 136, 1700, False, "f16"),   # 320 MB
    (20, 32, 8, 420, 420, True, "f16"),      # causal, four full rounds of short calls: four
    (1, 32, 8, 8192, 8192, True, "bf16"),    # of long ones: eight
], ids=lambda s: "x".join(map(str, s)))
def test_short_long_and_large(shape):
    B, Hq, Hkv, Nq, Nk, causal, dtype = shape
    gen = torch.Generator("cuda").manual_seed(Nk)
    dt = {"f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    q, k, v = (torch.randn(B, n, h, 64, generator=gen, device="cuda", dtype=dt)
               for n, h in ((Nq, Hq), (Nk, Hkv), (Nk, Hkv)))
    o, lse = fa.fwd(q, k, v, causal=causal, out_dtype=torch.float32)
    for slots in (4, 8):
        os, ls = fa.fwd(q, k, v, causal=causal, out_dtype=torch.float32, slots_per_workgroup=slots)
        assert torch.equal(o, os) and torch.equal(lse, ls)
