"""The fp32-weight attention kernel (fp32 inputs, and head sizes other than 64
and 128) at the edges of its blocks: 16 query columns and 16 keys a wave, 64,
32 or 16 keys a tile, columns padded to a multiple of 32.  Compared with the
fp64 oracle at the bound the suite holds fp32 arithmetic to (1e-4 on an fp32
result, helpers.check_against)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_18656_amd as fa
from paper_2608_18656_amd.inputs import DTYPES, make_qkv

from helpers import default_scale, to_np

pytestmark = pytest.mark.gpu

# B, Hq, Hkv, Nq, Nk, D, causal, dtype
SHAPES = [
    (1, 1, 1, 1, 1, 8, False, "f32"),
    (1, 2, 2, 15, 15, 24, True, "f32"),
    (2, 3, 1, 17, 33, 32, True, "f32"),
    (1, 4, 2, 16, 64, 64, False, "f32"),
    (1, 2, 2, 65, 65, 64, True, "f32"),
    (1, 5, 1, 31, 129, 128, True, "f32"),
    (1, 2, 1, 33, 47, 160, True, "f32"),
    (1, 1, 1, 130, 130, 256, True, "f32"),
    (3, 32, 1, 1, 100, 64, False, "f32"),       # decode: 32 heads share the keys, two column blocks
    (1, 4, 1, 63, 64, 40, True, "f16"),
    (2, 8, 2, 1, 257, 96, False, "bf16"),       # decode
    (1, 16, 1, 9, 200, 80, True, "f16"),        # a wave's 16 columns are one row's heads
    (1, 3, 3, 50, 79, 104, True, "bf16"),
    (1, 6, 2, 20, 20, 136, True, "f16"),
    (1, 2, 2, 49, 97, 192, False, "bf16"),
    (1, 4, 4, 18, 31, 224, True, "f16"),
    (1, 7, 1, 40, 66, 256, True, "bf16"),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_edges_against_oracle(shape):
    B, Hq, Hkv, Nq, Nk, D, causal, dtype = shape
    q, k, v = make_qkv(B, Hq, Hkv, Nq, Nk, D, dtype, seed=5000 + Nk + D)
    scale = default_scale(D)
    o, lse = fa.fwd(q.cuda(), k.cuda(), v.cuda(), causal=causal, scale=scale, out_dtype=torch.float32)
    o_ref, l_ref = oracle.attention(q, k, v, causal, scale)
    assert np.abs(to_np(o) - o_ref).max() <= 1e-4
    assert np.abs(to_np(lse) - l_ref).max() <= 1e-4
    if dtype != "f32":   # the shipped output is that result rounded once
        o16, _ = fa.fwd(q.cuda(), k.cuda(), v.cuda(), causal=causal, scale=scale)
        assert torch.equal(o16, o.to(DTYPES[dtype]))


@pytest.mark.parametrize("D,dtype", [(64, "f32"), (96, "bf16"), (256, "f16")])
def test_cache_lengths_and_rows_past_them(D, dtype):
    """Rows past a sequence's length hold NaN and are never used; an empty
    sequence, and rows of a chunk longer than its sequence, give 0 and -inf."""
    B, Hq, Hkv, Nq, Nk = 5, 6, 2, 20, 150
    lens = [150, 65, 16, 7, 0]
    q, k, v = make_qkv(B, Hq, Hkv, Nq, Nk, D, dtype, seed=77)
    scale = default_scale(D)
    for b, n in enumerate(lens):
        k[b, n:] = float("nan")
        v[b, n:] = float("nan")
    o, lse = fa.fwd_kvcache(q.cuda(), k.cuda(), v.cuda(), torch.tensor(lens, dtype=torch.int32).cuda(),
                            causal=True, scale=scale, out_dtype=torch.float32)
    for b, n in enumerate(lens):
        blind = max(0, Nq - n)   # rows that see no key
        assert torch.all(o[b, :blind] == 0) and torch.all(lse[b, :, :blind] == -float("inf"))
        if n:
            o_ref, l_ref = oracle.attention(q[b:b + 1, blind:], k[b:b + 1, :n], v[b:b + 1, :n], True, scale)
            assert np.abs(to_np(o[b:b + 1, blind:]) - o_ref).max() <= 1e-4
            assert np.abs(to_np(lse[b:b + 1, :, blind:]) - l_ref).max() <= 1e-4


@pytest.mark.parametrize("D,dtype", [(64, "f32"), (80, "f16"), (80, "bf16")])
def test_infinite_value_and_score(D, dtype):
    """An infinite value reaches its column alone; a score of -inf hides its key."""
    q, k, v = make_qkv(1, 2, 2, 33, 70, D, dtype, seed=9)
    scale = default_scale(D)
    v[0, 40, 0, 3] = float("inf")
    q[0, :, 1, 5] = 1.0
    k[0, 21, 1, 5] = -float("inf")
    o, lse = fa.fwd(q.cuda(), k.cuda(), v.cuda(), causal=False, scale=scale, out_dtype=torch.float32)
    assert torch.all(o[0, :, 0, 3] == float("inf"))
    v[0, 40, 0, 3] = 0.0
    keep = [j for j in range(70) if j != 21]
    o_ref, _ = oracle.attention(q, k.clone().nan_to_num(neginf=0.0), v, False, scale)
    o_hid, l_hid = oracle.attention(q[:, :, 1:], k[:, keep, 1:], v[:, keep, 1:], False, scale)
    cols = [d for d in range(D) if d != 3]
    assert np.abs(to_np(o)[0, :, 0][:, cols] - o_ref[0, :, 0][:, cols]).max() <= 1e-4
    assert np.abs(to_np(o)[0, :, 1] - o_hid[0, :, 0]).max() <= 1e-4
    assert np.abs(to_np(lse)[0, 1] - l_hid[0, 0]).max() <= 1e-4
