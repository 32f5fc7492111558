"""Scores and weights at the ends of their ranges in the fp32-weight attention
kernel, against the fp64 oracle at the bound the suite holds fp32 arithmetic to
(1e-4 on an fp32 result)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_18656_amd as fa

from helpers import to_np

pytestmark = pytest.mark.gpu

DTS = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}


def _against_oracle(q, k, v, scale, causal=False):
    o, lse = fa.fwd(q.cuda(), k.cuda(), v.cuda(), causal=causal, scale=scale, out_dtype=torch.float32)
    o_ref, l_ref = oracle.attention(q, k, v, causal, scale)
    assert np.abs(to_np(o) - o_ref).max() <= 1e-4
    assert np.abs(to_np(lse) - l_ref).max() <= 1e-4


@pytest.mark.parametrize("D", [32, 64, 96, 128, 160, 256])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_scores_from_the_last_columns(D, dtype):
    """All of a score comes from the last columns of D, that is from the last
    matrix product of its chain: a maximum of scores that lack it would set the
    base of the weights some 40 powers of two off."""
    if D in (64, 128) and dtype != "f32":
        pytest.skip("half-precision heads of 64 and 128 take another kernel")
    gen = torch.Generator().manual_seed(D)
    q, k = torch.zeros(1, 70, 4, D), torch.zeros(1, 300, 4, D)
    q[..., -4:] = 1.0
    k[..., -4:] = torch.randint(-7, 8, (1, 300, 4, 1), generator=gen).float()
    v = torch.randn(1, 300, 4, D, generator=gen)
    _against_oracle(*(t.to(DTS[dtype]) for t in (q, k, v)), 1.0)


@pytest.mark.parametrize("D,dtype", [(96, "f16"), (160, "f16"), (96, "bf16"), (64, "f32")])
@pytest.mark.parametrize("gap", [0.5, 8.5, 14.0, 17.0, 20.75, 24.25, 30.0, 40.0])
def test_values_on_keys_of_small_weight(D, dtype, gap):
    """One key outweighs the 1023 others by e^gap and has the value 0; the others'
    large values make up the result, so that their weights' own accuracy shows:
    at most 1024 products and as many additions, each within 2^-24, in each of
    the two sums that a result is the quotient of (2.5e-4 in the worst case; a
    weight of 16 bits is off by 2^-11 or more).  Every other row weighs all keys
    the same."""
    gen = torch.Generator().manual_seed(5)
    q, k = torch.zeros(1, 21, 2, D), torch.zeros(1, 1024, 2, D)
    q[:, ::2, :, 0] = 1.0
    k[0, 37, :, 0] = gap
    v = 3e4 + 3e4 * torch.rand(1, 1024, 2, D, generator=gen)
    v[0, 37] = 0.0
    q, k, v = (t.to(DTS[dtype]) for t in (q, k, v))
    o, lse = fa.fwd(q.cuda(), k.cuda(), v.cuda(), causal=False, scale=1.0, out_dtype=torch.float32)
    o_ref, l_ref = oracle.attention(q, k, v, False, 1.0)
    assert (np.abs(to_np(o) - o_ref) <= 2.5e-4 * np.abs(o_ref)).all()
    assert np.abs(to_np(lse) - l_ref).max() <= 1e-4


@pytest.mark.parametrize("D,dtype", [(96, "bf16"), (160, "bf16"), (64, "f32"), (192, "f32")])
@pytest.mark.parametrize("heavy", [2.625, 5.5])
def test_values_near_the_end_of_the_range(D, dtype, heavy):
    """The largest weight, seen late, belongs to a value of 2^126: weights above 1
    would take the product out of range."""
    q, k, v = (torch.zeros(1, n, 2, D) for n in (21, 300, 300))
    q[..., 0] = 1.0
    k[0, 290, :, 0] = heavy
    v[0, 290] = 2.0 ** 126
    q, k, v = (t.to(DTS[dtype]) for t in (q, k, v))
    o, _ = fa.fwd(q.cuda(), k.cuda(), v.cuda(), causal=False, scale=1.0, out_dtype=torch.float32)
    o_ref, _ = oracle.attention(q, k, v, False, 1.0)
    assert (np.abs(to_np(o) - o_ref) <= 2e-5 * o_ref).all()   # 300 additions within 2^-24 each


@pytest.mark.parametrize("D,dtype", [(64, "f32"), (192, "f32"), (96, "bf16"), (256, "bf16")])
@pytest.mark.parametrize("scale", [0.0, 1e-33, -2e-33])
def test_large_scores_of_a_tiny_scale(D, dtype, scale):
    """Products of q and k of up to some 10^34: a scale of 0 weighs all keys the
    same, one of 10^-33 leaves ordinary scores."""
    gen = torch.Generator().manual_seed(8)
    q, k, v = (torch.randn(1, n, 2, D, generator=gen) for n in (21, 150, 150))
    q, k, v = (t.to(DTS[dtype]) for t in (q * 1e16, k * 3e16 / D ** 0.5, v))
    _against_oracle(q, k, v, scale, causal=True)


@pytest.mark.parametrize("dtype,D,bound", [("f32", 64, 1.755e-7), ("f32", 128, 1.69e-7), ("bf16", 96, 1.27e-7)])
def test_exponents_near_zero(dtype, D, bound):
    """The heaviest weights' exponents lie near 0, where fp32 holds them best: the
    mean error (2-norm) against fp64 over eight seeds, 1.70e-7, 1.62e-7 and
    1.18e-7, stays below half the way to what exponents shifted by 4 give (1.81e-7,
    1.76e-7 and 1.36e-7)."""
    errs = []
    for seed in range(8):
        gen = torch.Generator("cuda").manual_seed(seed)
        q, k, v = (torch.randn(1, n, 4, D, generator=gen, device="cuda").to(DTS[dtype]) for n in (400, 400, 400))
        o, _ = fa.fwd(q, k, v, causal=True, out_dtype=torch.float32)
        s = torch.matmul(q[0].transpose(0, 1).double().contiguous(), k[0].permute(1, 2, 0).double().contiguous()) / D ** 0.5
        s.masked_fill_(torch.ones(400, 400, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
        ref = torch.matmul(torch.softmax(s, -1), v[0].transpose(0, 1).double().contiguous()).transpose(0, 1)
        errs.append(((o[0].double() - ref).norm() / ref.norm()).item())
    assert sum(errs) / 8 < bound
