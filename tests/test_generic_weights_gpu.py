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
