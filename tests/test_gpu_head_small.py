"""The dense head on small and unaligned shapes: one to many 32 x 32 tiles, part of a tile in both directions,
contractions shorter than a wave's first step and not a multiple of it, rows at 16-, 4- and 2-byte alignment,
one to several chunks of the dX contraction, and sizes on both sides of the large-tile kernels' rules."""
import pytest

import synth
from gpu_helpers import rel_err, say
from test_gpu_any import SUM_TOL, close_bf16, ref_positives

pytestmark = pytest.mark.gpu

# B, F_s, H
SHAPES = [(1, 1, 1), (77, 500, 1003), (33, 37, 65), (8, 768, 1024), (32, 512, 24), (40, 770, 300), (100, 63, 4001), (5, 16, 31),
          (300, 384, 1001), (31, 768, 16384),
          # past the direct kernel's limits: dX by its work, dW of few rows, logits of odd rows
          (77, 768, 16387), (16, 301, 4098), (900, 559, 1935)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("bias", [False, True])
def test_head(shape, bias):
    import torch
    import paper_2606_01117_amd as hs
    B, F_s, H = shape
    say("head", shape, bias)
    gen = torch.Generator(device="cuda").manual_seed(6)
    X = torch.randn((B, F_s), device="cuda", generator=gen).bfloat16()
    W = (torch.randn((H, F_s), device="cuda", generator=gen) / F_s ** 0.5).bfloat16()
    b = torch.randn(H, device="cuda", generator=gen) if bias else None
    pos = torch.randint(-1, H + 1, (B, 7), dtype=torch.int32, device="cuda", generator=gen)
    bf = synth.DT_BF16
    Y, dY = (torch.empty((B, H), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    hs.haste_head_fwd(B, F_s, H, bf, X, W, b, Y)
    z = X.double() @ W.double().t() + (b.double() if bias else 0.0)
    assert close_bf16(Y, z, float(z.abs().max()))
    hs.haste_head_fwd_bce(B, F_s, H, bf, X, W, b, pos, dY)
    if F_s % 8 or H % 8:                          # that of the rounded logits, bit for bit
        dY2 = torch.empty_like(Y)
        hs.haste_bce_grad(B, H, bf, Y, pos, dY2)
        assert torch.equal(dY.view(torch.int16), dY2.view(torch.int16))
    assert rel_err(dY.cpu().float(), (torch.sigmoid(z) - ref_positives(pos, H)).cpu()) < 2e-2
    dW, dX = torch.empty((H, F_s), device="cuda"), torch.ones((B, F_s), device="cuda")
    ws = hs.workspace(hs.haste_head_workspace_bytes(B, F_s, H, bf))
    ws.fill_(0xff)
    hs.haste_head_bwd(B, F_s, H, bf, X, W, dY, dW, dX, 1, ws)
    assert rel_err(dW.cpu(), (dY.double().t() @ X.double()).cpu()) < SUM_TOL
    assert rel_err(dX.cpu(), (dY.double() @ W.double() + 1.0).cpu()) < SUM_TOL
