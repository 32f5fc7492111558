"""The fp32-weight attention kernel in each of its layouts (column blocks, key
parts; which one runs depends on the grid), with offsets past a buffer view's
31 bits, and where its weights are special: bases that move in every tile,
weights that leave the range of one 16-bit term, scales of either sign.  fp64
reference; the bound is the one the suite holds fp32 arithmetic to (1e-4 on an
fp32 result)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_18656_amd as fa
from paper_2608_18656_amd.inputs import make_qkv

from helpers import default_scale, to_np

pytestmark = pytest.mark.gpu

# B, Hq, Hkv, Nq, Nk, D, causal, dtype: more columns than the small layouts take
SHAPES = [
    (3, 180, 180, 17, 40, 24, False, "f16"),     # (4, 2)
    (1, 540, 270, 20, 70, 96, True, "bf16"),
    (3, 180, 180, 30, 33, 88, True, "f16"),      # (2, 2): causal, about square
    (1, 260, 260, 70, 70, 96, True, "bf16"),
    (2, 300, 300, 17, 40, 64, False, "f32"),     # (2, 4)
    (1, 33, 33, 250, 97, 192, False, "f32"),     # (4, 2)
    (1, 130, 130, 100, 37, 136, False, "f32"),   # (2, 2), as in every fp32 call of 129 to 160 columns
    (1, 300, 300, 140, 150, 160, True, "f32"),
    (2, 130, 130, 17, 33, 192, False, "bf16"),   # (8, 1)
    (1, 260, 260, 129, 140, 256, True, "f16"),
    (2, 130, 130, 130, 130, 224, True, "f32"),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_large_grids(shape):
    B, Hq, Hkv, Nq, Nk, D, causal, dtype = shape
    q, k, v = make_qkv(B, Hq, Hkv, Nq, Nk, D, dtype, seed=6000 + Nk + D)
    scale = default_scale(D)
    o, lse = fa.fwd(q.cuda(), k.cuda(), v.cuda(), causal=causal, scale=scale, out_dtype=torch.float32)
    o_ref, l_ref = oracle.attention(q, k, v, causal, scale)
    assert np.abs(to_np(o) - o_ref).max() <= 1e-4
    assert np.abs(to_np(lse) - l_ref).max() <= 1e-4


@pytest.mark.parametrize("dtype,Nk", [(torch.float16, 33), (torch.float32, 17)])
def test_key_rows_of_64_mib_and_more(dtype, Nk):
    """A tile's last key row starts 2 GiB or more after its first."""
    H, D = 131073, 256
    gen = torch.Generator("cuda").manual_seed(3)
    q, k, v = (torch.randn(1, n, H, D, generator=gen, device="cuda", dtype=torch.float32).to(dtype) for n in (1, Nk, Nk))
    o, _ = fa.fwd(q, k, v, scale=default_scale(D), out_dtype=torch.float32)
    for h0 in range(0, H, 16384):
        h = slice(h0, min(h0 + 16384, H))
        w = torch.softmax((q[0, :, h].double() * k[0, :, h].double()).sum(-1) * default_scale(D), 0)
        ref = (w[:, :, None] * v[0, :, h].double()).sum(0)
        assert (o[0, 0, h].double() - ref).abs().max().item() <= 1e-4


@pytest.mark.parametrize("D,dtype", [(64, "f32"), (96, "bf16"), (96, "f16"), (200, "f16")])
@pytest.mark.parametrize("scale", [0.3, -0.2, 0.0])
def test_rising_scores_and_scales(D, dtype, scale):
    """Keys grow along the sequence: each tile raises the rows' maxima."""
    q, k, v = make_qkv(1, 4, 2, 40, 300, D, dtype, seed=11)
    k = (k.float() * torch.linspace(0.1, 4, 300)[None, :, None, None]).to(k.dtype)
    o, lse = fa.fwd(q.cuda(), k.cuda(), v.cuda(), causal=True, scale=scale, out_dtype=torch.float32)
    o_ref, l_ref = oracle.attention(q, k, v, True, scale)
    assert np.abs(to_np(o) - o_ref).max() <= 1e-4
    assert np.abs(to_np(lse) - l_ref).max() <= 1e-4


@pytest.mark.parametrize("D,dtype", [(96, "f16"), (96, "bf16"), (160, "f16"), (64, "f32")])
def test_tiny_weights(D, dtype):
    """One key carries weight 1, the others 2^-46 each: an infinite value among
    those still shows, and the one key's value counts whole."""
    dt = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    q = torch.zeros(1, 16, 1, D, dtype=dt)
    k = torch.zeros(1, 100, 1, D, dtype=dt)
    v = torch.zeros(1, 100, 1, D, dtype=dt)
    q[..., 0] = 1.0
    k[0, 37, 0, 0] = 32.0      # score 32 against 0: weights e^-32 = 2^-46.2
    v[0, 5, 0, 3] = float("inf")
    v[0, 80, 0, 4] = -float("inf")
    v[0, 37, 0, 6] = 1.5
    o = to_np(fa.fwd(q.cuda(), k.cuda(), v.cuda(), causal=False, scale=1.0, out_dtype=torch.float32)[0])
    assert np.all(o[..., 3] == np.inf) and np.all(o[..., 4] == -np.inf)
    assert np.abs(o[..., 6] - 1.5).max() <= 1e-6
    assert np.all(np.delete(o, [3, 4, 6], axis=-1) == 0)
