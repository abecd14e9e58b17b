"""Layers of any group size, support width, feature width and label count against dense fp64 products
on the GPU: the shapes at which the kernels for them change (tiles, remainders, access widths)."""
import pytest

import synth
from gpu_helpers import rel_err, say

pytestmark = pytest.mark.gpu

# fp32 sums of bf16 products: each of the n terms and the partial sums round by at most 2^-24 of the
# running sum, which random signs keep within sqrt(n) of a term; 2e-5 of the largest entry covers
# n = 2^16 with a margin of ten
SUM_TOL = 2e-5

# B, F_s, L, G, F_in: rows in one 32- or 64-row tile and past it; F_s at and past the tiles of 512 and
# 768 features and the two shares of wider inputs; supports of one slot pair to all features; groups
# packed by 1, 2, 4, 8 labels in one write; label counts that end inside a step, odd and even
SHAPES = [
    (32, 768, 640, 1, 64), (33, 768, 1027, 1, 63), (64, 512, 514, 2, 100), (65, 513, 516, 4, 256),
    (7, 300, 24 * 43, 24, 48), (77, 500, 24 * 131, 24, 48), (130, 896, 35 * 30, 35, 181), (96, 769, 992, 32, 256),
    (40, 640, 333, 3, 1), (16, 65, 8 * 37, 8, 65), (70, 768, 16 * 81, 16, 200), (300, 384, 2048, 64, 256),
    (48, 905, 1001, 7, 255), (1, 256, 1, 1, 2), (64, 768, 260, 260, 33), (33, 768, 602, 14, 129),
    (100, 766, 4100, 4, 31),
]


def layer(shape, seed=0):
    import torch
    B, F_s, L, G, F_in = shape
    gen = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *s: torch.randn(s, device="cuda", generator=gen)
    idx = torch.rand((L // G, F_s), device="cuda", generator=gen).argsort(1)[:, :F_in].sort(1).values.int().contiguous()
    X, W, dY = r(B, F_s).bfloat16(), (r(L, F_in) / F_in ** 0.5).bfloat16(), r(B, L).bfloat16()
    sup = idx.long().repeat_interleave(G, 0)
    Wd = torch.zeros((L, F_s), dtype=torch.float64, device="cuda").scatter_(1, sup, W.double())
    return X, idx, W, dY, sup, Wd


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("beta", [0, 1])
def test_bwd_x(shape, beta):
    import torch
    import paper_2606_01117_amd as hs
    B, F_s, L, G, F_in = shape
    say("bwd_x", shape, beta)
    X, idx, W, dY, sup, Wd = layer(shape)
    desc = hs.make_desc(B, F_s, L, G, F_in, synth.DT_BF16)
    ws = hs.workspace(hs.haste_workspace_bytes(desc, hs.HASTE_OP_BWD_X))
    ws.fill_(0xff)
    dX = torch.ones((B, F_s), device="cuda")
    hs.haste_bwd_x(desc, idx, W, dY, dX, beta, ws)
    ref = dY.double() @ Wd + beta
    assert rel_err(dX.cpu(), ref.cpu()) < SUM_TOL
