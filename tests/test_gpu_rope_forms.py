"""The rotary embedding's two forms (angles shared by the heads of a token for
head dims that are a multiple of 16, one angle per pair otherwise) at the edges
of their tiles: one token, partial groups of four tokens, one head and more
heads than a workgroup preloads, the smallest and largest head dims, far
positions, in place, and backward as the inverse.

Tolerance: the angle is exact to fp32 (2^-24 of pi), then one bf16 rounding:
2^-8 of the pair's length is twice that."""
import sys

import pytest

pytestmark = pytest.mark.gpu

CASES = [(1, 1, 16, 0), (3, 40, 128, 131000), (4, 8, 64, 7), (5, 3, 256, 1), (9, 70, 128, 28672),
         (6, 2, 10, 3), (2, 5, 24, 900), (257, 32, 128, 0)]


@pytest.mark.parametrize("tokens,heads,d,pos0", CASES)
def test_rope_forms(gpu, tokens, heads, d, pos0):
    import torch
    from paper_2606_01143_amd import binding as B
    sys.stderr.write(f"\n[gpu-case] rope tokens={tokens} heads={heads} d={d} pos0={pos0}\n")
    sys.stderr.flush()
    theta = 500000.0
    g = torch.Generator().manual_seed(1)
    x = torch.randn(tokens, heads, d, generator=g).to(torch.bfloat16)
    pos = torch.arange(pos0, pos0 + tokens, dtype=torch.float64)
    ang = pos[:, None] * theta ** (-2.0 * torch.arange(d // 2, dtype=torch.float64) / d)
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = x.double()[..., :d // 2], x.double()[..., d // 2:]
    size = (a * a + b * b).sqrt().repeat(1, 1, 2)
    xd = x.cuda()
    for sign, call in ((1.0, B.rope_fwd), (-1.0, B.rope_bwd)):
        want = torch.cat([a * c - sign * b * s, b * c + sign * a * s], -1)
        y = torch.full_like(xd, float("nan"))
        call(xd, y, pos0, theta)
        inplace = xd.clone()
        call(inplace, inplace, pos0, theta)
        torch.cuda.synchronize()
        assert torch.equal(y, inplace)
        assert bool(((y.cpu().double() - want).abs() <= 2.0 ** -8 * size + 1e-30).all())
