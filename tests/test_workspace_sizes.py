"""A decode workspace sized for a cache serves every shorter cache (a program
sizes it once, for its longest): fa_workspace_bytes never falls as Nk grows,
though the split count may."""
import random

import pytest
import torch

import paper_2608_18656_amd as fa
from paper_2608_18656_amd import workspace_bytes


@pytest.mark.parametrize("D", [64, 128])
def test_size_never_falls_as_the_cache_grows(D):
    rng = random.Random(D)
    shapes = [(1, 32, 32), (16, 32, 8), (4, 32, 8), (8, 16, 16), (54, 4, 1), (3, 12, 3), (56, 4, 1), (1, 24, 3)]
    shapes += [(rng.randint(1, 80), g * h, h) for h in (1, 2, 3, 6, 12, 40) for g in (1, 4, 17)]
    for B, Hq, Hkv in shapes:
        lengths = sorted([*range(1, 33000, 509), *(int(2 ** rng.uniform(5, 30.9)) for _ in range(60))])
        sizes = [workspace_bytes(B, Hq, Hkv, 1, n, D, "bf16") for n in lengths]
        assert sizes == sorted(sizes), (B, Hq, Hkv)
        assert sizes[0] >= B * Hq * (D + 2) * 4


@pytest.mark.gpu
def test_shorter_caches_fit_what_the_longest_was_given():
    """64 x 16/1 heads, D = 64: 16448 keys take four splits, 3264 take eight; with
    a workspace of the caller's, and with the library's while the stream is
    captured (when none can be allocated)."""
    B, Hq, Hkv, D = 64, 16, 1, 64
    gen = torch.Generator("cuda").manual_seed(6)
    q = torch.randn(B, 1, Hq, D, generator=gen, device="cuda", dtype=torch.float16)
    long, short = (tuple(torch.randn(B, n, Hkv, D, generator=gen, device="cuda", dtype=torch.float16) for _ in range(2))
                   for n in (16448, 3264))
    ws = torch.empty(workspace_bytes(B, Hq, Hkv, 1, 16448, D, "f16"), dtype=torch.uint8, device="cuda")
    ref, _ = fa.fwd(q, *short, num_splits=8)
    assert torch.equal(fa.fwd(q, *short, workspace=ws)[0], ref)
    out = torch.zeros_like(q)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        fa.fwd(q, *long, out=out)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            fa.fwd(q, *short, out=out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
