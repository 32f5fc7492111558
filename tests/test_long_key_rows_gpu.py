"""Key rows (all key/value heads of one position) so long that a tile of them
passes 2 GiB, where the prefill and decode kernels' 32-bit offsets end: which
kernels such calls take, on the CPU, and their results against fp64."""
import pytest
import torch

import paper_2608_18656_amd as fa

from helpers import default_scale

# most heads whose 32 key rows (decode) stay below 2 GiB
LAST = {64: 541200, 128: 270600}


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
def test_decode_takes_no_splits_past_2_gib(D, dtype):
    H = LAST[D]
    assert 31 * H * D * 2 + 2 * D <= 2**31 - 1 < 31 * (H + 1) * D * 2 + 2 * D
    assert fa.workspace_bytes(1, H, H, 1, 32, D, dtype) == H * (D + 2) * 4
    assert fa.workspace_bytes(1, H + 1, H + 1, 1, 32, D, dtype) == 0
    assert fa.workspace_bytes(3, 4 * H + 4, H + 1, 1, 4096, D, dtype, 7) == 0


def _check(q, k, v, o, causal):
    """o [1, Nq, H, D] against fp64, 16384 heads at a time, within 2e-3 (the suite's
    bound for fp16 / bf16 inputs)."""
    D, Nq, Nk = q.shape[3], q.shape[1], k.shape[1]
    for h0 in range(0, q.shape[2], 16384):
        h = slice(h0, h0 + 16384)
        for i in range(Nq):
            n = Nk - Nq + i + 1 if causal else Nk
            w = torch.softmax((q[0, i, h].double() * k[0, :n, h].double()).sum(-1) * default_scale(D), 0)
            ref = (w[:, :, None] * v[0, :n, h].double()).sum(0)
            assert (o[0, i, h].double() - ref).abs().max().item() <= 2e-3, (h0, i)


@pytest.mark.gpu
@pytest.mark.parametrize("D,H,Nq,Nk,dtype", [
    (128, LAST[128], 1, 33, "f16"),          # the last size the decode kernel takes
    (128, LAST[128] + 1, 1, 33, "bf16"),
    (128, 541201, 1, 40, "f16"),             # 32 rows reach 4 GiB
    (64, 1082402, 1, 33, "f16"),
    (128, LAST[128] + 1, 3, 40, "f16"),      # prefill, tiles of 32 keys
    (64, 270600, 2, 65, "bf16"),             # and of 64
])
def test_contiguous(D, H, Nq, Nk, dtype):
    dt = {"f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    gen = torch.Generator("cuda").manual_seed(3)
    q, k, v = (torch.randn(1, n, H, D, generator=gen, device="cuda", dtype=dt) for n in (Nq, Nk, Nk))
    o, lse = fa.fwd(q, k, v, causal=True, out_dtype=torch.float32)
    _check(q, k, v, o, True)
    full = torch.tensor([Nk], dtype=torch.int32, device="cuda")
    oc, lc = fa.fwd_kvcache(q, k, v, full, causal=True, out_dtype=torch.float32)
    assert torch.equal(oc, o) and torch.equal(lc, lse)


@pytest.mark.gpu
@pytest.mark.parametrize("D,H,Nq", [(128, LAST[128] + 1, 1), (128, LAST[128] + 1, 5), (64, 270601, 3)])
def test_paged(D, H, Nq):
    """Two sequences in three pages of 64 keys, one page shared, equal the gathered cache bit for bit."""
    gen = torch.Generator("cuda").manual_seed(4)
    kp, vp = (torch.randn(3, 64, H, D, generator=gen, device="cuda", dtype=torch.float16) for _ in range(2))
    q = torch.randn(2, Nq, H, D, generator=gen, device="cuda", dtype=torch.float16)
    table = torch.tensor([[2, 0], [1, 2]], dtype=torch.int32, device="cuda")
    lens = torch.tensor([90, 64], dtype=torch.int32, device="cuda")
    o, lse = fa.fwd_kvcache_paged(q, kp, vp, table, lens, causal=True, out_dtype=torch.float32)
    for b, pages in enumerate(table.tolist()):
        kc, vc = (torch.cat([t[i] for i in pages])[None] for t in (kp, vp))
        oc, lc = fa.fwd_kvcache(q[b:b + 1], kc, vc, lens[b:b + 1], causal=True, out_dtype=torch.float32)
        assert torch.equal(oc, o[b:b + 1]) and torch.equal(lc, lse[b:b + 1])
        n = int(lens[b])
        _check(q[b:b + 1], kc[:, :n], vc[:, :n], oc, True)
