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
    # as large as the forward's and backward-weight's rules ask for: odd supports in packs of 8, one label, few slots
    (64, 700, 8 * 137, 8, 65), (64, 768, 1, 1, 255), (300, 766, 4100, 4, 31), (64, 511, 1500, 3, 100),
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


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("beta", [0, 1])
def test_bwd_w(shape, beta):
    import torch
    import paper_2606_01117_amd as hs
    B, F_s, L, G, F_in = shape
    say("bwd_w", shape, beta)
    X, idx, W, dY, sup, Wd = layer(shape, 1)
    desc = hs.make_desc(B, F_s, L, G, F_in, synth.DT_BF16)
    need = hs.haste_workspace_bytes(desc, hs.HASTE_OP_BWD_W)
    ws = hs.workspace(need)
    if ws is not None:
        ws.fill_(0xff)
    dW, db = torch.ones((L, F_in), device="cuda"), torch.ones(L, device="cuda")
    hs.haste_bwd_w(desc, X, idx, dY, dW, db, beta, ws)
    ref = (dY.double().t() @ X.double()).gather(1, sup) + beta
    assert rel_err(dW.cpu(), ref.cpu()) < SUM_TOL
    assert rel_err(db.cpu(), (dY.double().sum(0) + beta).cpu()) < SUM_TOL


def ref_positives(pos, L):
    import torch
    T = torch.zeros((pos.shape[0], L), dtype=torch.float64, device="cuda")
    rows = torch.arange(pos.shape[0], device="cuda")[:, None].expand_as(pos)
    ok = (pos >= 0) & (pos < L)
    T[rows[ok], pos[ok].long()] = 1.0
    return T


def close_bf16(a, ref, scale):
    """Within one rounding to bf16 of the 64-bit value (half an ulp, 2^-8 of it, and as much again where
    the fp32 sum lies at the tie), beside the fp32 sum's own error."""
    return bool(((a.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + SUM_TOL * scale).all())


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("bias", [False, True])
def test_fwd(shape, bias):
    import torch
    import paper_2606_01117_amd as hs
    B, F_s, L, G, F_in = shape
    say("fwd", shape, bias)
    X, idx, W, _, sup, Wd = layer(shape, 2)
    b = torch.randn(L, device="cuda") if bias else None
    desc = hs.make_desc(B, F_s, L, G, F_in, synth.DT_BF16)
    Y = torch.full((B, L), 7.0, dtype=torch.bfloat16, device="cuda")
    hs.haste_fwd(desc, X, idx, W, b, Y)
    ref = X.double() @ Wd.t() + (b.double() if bias else 0.0)
    assert close_bf16(Y, ref, float(ref.abs().max()))
    # the loss gradient: that of the rounded logits, bit for bit, and backward-weight on it
    pos = torch.randint(-2, L + 2, (B, 9), dtype=torch.int32, device="cuda")
    dY, dY2, dW = torch.empty_like(Y), torch.empty_like(Y), torch.empty((L, F_in), device="cuda")
    ws = hs.workspace(hs.haste_workspace_bytes(desc, hs.HASTE_OP_FWD_BCE))
    if ws is not None:
        ws.fill_(0xff)
    hs.haste_fwd_bce(desc, X, idx, W, b, pos, dY, dW, None, 0, ws)
    T = ref_positives(pos, L)
    if G % 16 or F_in not in (32, 64, 128):       # the fused kernel's gradient is that of the fp32 logits
        hs.haste_bce_grad(B, L, synth.DT_BF16, Y, pos, dY2)
        assert torch.equal(dY.view(torch.int16), dY2.view(torch.int16))
    assert rel_err(dY.cpu().float(), (torch.sigmoid(ref) - T).cpu()) < 2e-2
    refw = (dY.double().t() @ X.double()).gather(1, sup)
    assert rel_err(dW.cpu(), refw.cpu()) < SUM_TOL


@pytest.mark.parametrize("shape", [(33, 768, 1027, 1, 63), (77, 500, 24 * 131, 24, 48), (130, 768, 1050, 35, 181)])
def test_fwd_not_finite(shape):
    """An infinity or a NaN in X reaches the labels whose support holds its feature, and no others."""
    import torch
    import paper_2606_01117_amd as hs
    B, F_s, L, G, F_in = shape
    say("fwd_not_finite", shape)
    X, idx, W, _, sup, Wd = layer(shape, 3)
    X[B - 1, 5] = float("inf")
    X[B // 2, F_s - 1] = float("nan")
    desc = hs.make_desc(B, F_s, L, G, F_in, synth.DT_BF16)
    Y = torch.empty((B, L), dtype=torch.bfloat16, device="cuda")
    hs.haste_fwd(desc, X, idx, W, None, Y)
    touched = torch.zeros((B, L), dtype=torch.bool, device="cuda")
    touched[B - 1] |= (sup == 5).any(1)
    touched[B // 2] |= (sup == F_s - 1).any(1)
    assert torch.equal(~torch.isfinite(Y), touched)
    ref = torch.where(torch.isfinite(X), X, 0).double() @ Wd.t()
    assert close_bf16(torch.where(touched, 0, Y.double()), torch.where(touched, 0, ref), float(ref.abs().max()))


# groups that the accumulator kernel took (16 and 32 labels), any other group, odd widths and labels, two feature
# shares, and both widths of 64-row tiles; 32- and 64-row tiles, and a segment of more than one step
@pytest.mark.parametrize("shape", [(64, 768, 32 * 150, 32, 64), (70, 768, 16 * 81, 16, 200), (33, 768, 1027, 1, 63), (20, 300, 24 * 131, 24, 48),
                                   (130, 896, 35 * 30, 35, 181), (300, 384, 2048, 64, 256), (128, 768, 4096, 4, 64)])
def test_bwd_x_not_finite(shape):
    """An infinity or a NaN in dY reaches the features of its label's support, and no others: one element, several
    of a row in one group and in several, both infinities at once, an infinity that meets a zero weight and
    one that meets infinite weights, the last row and label, and a whole row."""
    import torch
    import paper_2606_01117_amd as hs
    B, F_s, L, G, F_in = shape
    say("bwd_x_not_finite", shape)
    X, idx, W, dY, sup, Wd = layer(shape, 8)
    inf, nan = float("inf"), float("nan")
    W[L // 3, F_in // 2] = 0.0
    Wd[L // 3, sup[L // 3, F_in // 2]] = 0.0
    li = L // 4
    W[li, 0], W[li, F_in - 1] = inf, -inf
    Wd[li] = 0.0                                  # (its products are added below)
    for b, l, v in [(3, 0, inf), (3, 1, inf), (3, L // 2, -inf), (B // 2, L // 3, -inf), (B - 1, L - 1, nan), (B - 1, 5, inf), (2, li, -inf)]:
        dY[b, l] = v
    dY[7] = nan
    desc = hs.make_desc(B, F_s, L, G, F_in, synth.DT_BF16)
    ws = hs.workspace(hs.haste_workspace_bytes(desc, hs.HASTE_OP_BWD_X))
    ws.fill_(0xff)
    dX = torch.ones((B, F_s), device="cuda")
    hs.haste_bwd_x(desc, idx, W, dY, dX, 1, ws)
    bad = ~torch.isfinite(dY)
    ref = torch.where(bad, 0, dY).double() @ Wd + 1.0
    assert bool((dY[:, li] != 0).all())
    for b, l in bad.nonzero().tolist() + [(b, li) for b in range(B) if b != 2]:
        if b != 7:
            ref[b, sup[l]] += dY[b, l].double() * W[l].double()
    ref[7, sup.unique()] = nan
    assert torch.equal(torch.isnan(dX), torch.isnan(ref)) and torch.equal(torch.isinf(dX), torch.isinf(ref))
    assert torch.equal(dX[torch.isinf(ref)] > 0, ref[torch.isinf(ref)] > 0)
    ok = torch.isfinite(ref)
    assert rel_err(torch.where(ok, dX, 0).cpu(), torch.where(ok, ref, 0).cpu()) < SUM_TOL


# fp32: one unit, part of one, several per group; 64-slot chunks, part of one and four; F_s past 512 and
# 768; aligned and odd labels and supports; batches of part of a row tile, and of several slabs
SHAPES_F32 = [
    (32, 256, 4096, 8, 32), (128, 768, 2048, 16, 64), (33, 768, 1027, 1, 63), (65, 513, 516, 4, 256), (77, 500, 24 * 131, 24, 48),
    (130, 896, 35 * 30, 35, 181), (40, 640, 333, 3, 1), (300, 384, 2048, 64, 128), (1, 65, 1, 1, 2), (17, 905, 602, 14, 100),
    (64, 768, 260, 260, 33), (16, 768, 16 * 300, 16, 65),
    # as many groups as backward-feature's rule asks for, three chunks of odd supports
    (130, 896, 35 * 120, 35, 181),
]


def layer_f32(shape, seed):
    import torch
    B, F_s, L, G, F_in = shape
    gen = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *s: torch.randn(s, device="cuda", generator=gen)
    idx = torch.rand((L // G, F_s), device="cuda", generator=gen).argsort(1)[:, :F_in].sort(1).values.int().contiguous()
    sup = idx.long().repeat_interleave(G, 0)
    return r(B, F_s), idx, r(L, F_in) / F_in ** 0.5, r(B, L), r(L), sup


@pytest.mark.parametrize("shape", SHAPES_F32)
@pytest.mark.parametrize("beta", [0, 1])
def test_f32(shape, beta):
    """fp32 sums of fp32 products: n terms, each product and partial sum rounded to 2^-24 of itself; random
    signs keep the error within 3 sqrt(n) 2^-24 of a term's size, under 1e-5 of the largest entry."""
    import torch
    import paper_2606_01117_amd as hs
    B, F_s, L, G, F_in = shape
    say("f32", shape, beta)
    X, idx, W, dY, bias, sup = layer_f32(shape, 4)
    desc = hs.make_desc(B, F_s, L, G, F_in, synth.DT_F32)
    dense = torch.zeros((L, F_s), dtype=torch.float64, device="cuda").scatter_(1, sup, W.double())
    Y = torch.empty((B, L), device="cuda")
    for b in (None, bias):
        hs.haste_fwd(desc, X, idx, W, b, Y)
        assert rel_err(Y.cpu(), (X.double() @ dense.t() + (0 if b is None else b.double())).cpu()) < 1e-5
    dW, db = torch.ones((L, F_in), device="cuda"), torch.ones(L, device="cuda")
    hs.haste_bwd_w(desc, X, idx, dY, dW, db, beta, hs.workspace(hs.haste_workspace_bytes(desc, hs.HASTE_OP_BWD_W)))
    assert rel_err(dW.cpu(), ((dY.double().t() @ X.double()).gather(1, sup) + beta).cpu()) < 1e-5
    assert rel_err(db.cpu(), (dY.double().sum(0) + beta).cpu()) < 1e-5
    ws = hs.workspace(hs.haste_workspace_bytes(desc, hs.HASTE_OP_BWD_X))
    ws.fill_(0xff)
    dX = torch.ones((B, F_s), device="cuda")
    hs.haste_bwd_x(desc, idx, W, dY, dX, beta, ws)
    assert rel_err(dX.cpu(), (dY.double() @ dense + beta).cpu()) < 1e-5


def test_f32_not_finite():
    """An infinity in X or dY reaches the outputs the definition names, and no others."""
    import torch
    import paper_2606_01117_amd as hs
    shape = B, F_s, L, G, F_in = (33, 300, 24 * 40, 24, 50)
    X, idx, W, dY, _, sup = layer_f32(shape, 5)
    desc = hs.make_desc(B, F_s, L, G, F_in, synth.DT_F32)
    Xi, Yi = X.clone(), dY.clone()
    Xi[7, 11] = float("inf")
    Yi[5, 100] = float("inf")
    Y, dW, dX = torch.empty((B, L), device="cuda"), torch.empty((L, F_in), device="cuda"), torch.empty((B, F_s), device="cuda")
    hs.haste_fwd(desc, Xi, idx, W, None, Y)
    bad = torch.zeros((B, L), dtype=torch.bool, device="cuda")
    bad[7] = (sup == 11).any(1)
    assert torch.equal(~torch.isfinite(Y), bad)
    hs.haste_bwd_w(desc, Xi, idx, dY, dW, None, 0, None)
    assert torch.equal(~torch.isfinite(dW), sup == 11)
    hs.haste_bwd_x(desc, idx, W, Yi, dX, 0, hs.workspace(hs.haste_workspace_bytes(desc, hs.HASTE_OP_BWD_X)))
    bad = torch.zeros((B, F_s), dtype=torch.bool, device="cuda")
    bad[5, sup[100]] = True
    assert torch.equal(~torch.isfinite(dX), bad)


# layers whose queried workspace grew with these kernels: shape, dtype, and the bytes that the calls
# (haste_bwd_x, haste_tail_step, haste_tail_step_sgd) took before, which they still take
SCRATCH = [
    ((128, 512, 55848, 8, 128), synth.DT_BF16, (16777216, 17039616, 45633792)),
    ((64, 384, 36396, 4, 128), synth.DT_BF16, (12582912, 12697856, 31332608)),
    ((33, 768, 114792, 8, 15), synth.DT_BF16, (50331904, 50331904, 57219584)),
    ((256, 256, 24880, 2, 256), synth.DT_BF16, (16777472, 16777472, 42254592)),
    ((128, 298, 60816, 16, 256), synth.DT_BF16, (19529984, 19529984, 81805568)),
    ((1, 384, 436416, 32, 128), synth.DT_F32, (25166080, 25166080, 248611072)),
    # an odd number of 32-row tiles, whose partials are then fewer than 8 segments of 64-row tiles
    ((1030, 768, 65536, 4, 128), synth.DT_BF16, (25952256, 28629248, 62183680)),
    ((65, 768, 512, 4, 128), synth.DT_BF16, (2359296, 2573568, 2835712)),
]


@pytest.mark.parametrize("shape,dtype,least", SCRATCH)
def test_scratch_limits(shape, dtype, least):
    """With the smaller workspace: the results of the queried one (in another order of the fp32 sums, by another
    kernel or with fewer segments), and not a byte written behind it."""
    import torch
    import paper_2606_01117_amd as hs
    B, F_s, L, G, F_in = shape
    f32 = dtype == synth.DT_F32
    say("scratch", shape, dtype)
    gen = torch.Generator(device="cuda").manual_seed(6)
    r = lambda *s: torch.randn(s, device="cuda", generator=gen)
    cast = (lambda t: t) if f32 else (lambda t: t.bfloat16())
    idx = torch.rand((L // G, F_s), device="cuda", generator=gen).argsort(1)[:, :F_in].sort(1).values.int().contiguous()
    X, W, dY0, m0 = cast(r(B, F_s)), cast(r(L, F_in) / F_in ** 0.5), cast(r(B, L)), r(L, F_in)
    pos = torch.randint(0, L, (B, 5), device="cuda", generator=gen).int()
    desc = hs.make_desc(B, F_s, L, G, F_in, dtype)
    opt = hs.sgd_opts(0.1, 0.9, 1e-4)

    def bwd_x(ws):
        dX = torch.ones((B, F_s), device="cuda")
        hs.haste_bwd_x(desc, idx, W, dY0, dX, 1, ws)
        return [dX]

    def step(ws):
        dY, dW, dX = torch.empty_like(dY0), torch.empty_like(m0), torch.empty((B, F_s), device="cuda")
        hs.haste_tail_step(desc, X, idx, W, None, pos, dY, dW, None, 0, dX, 0, ws)
        return [dY.float(), dW, dX]

    def sgd(ws):
        dY, m, dX, Wn = torch.empty_like(dY0), m0.clone(), torch.empty((B, F_s), device="cuda"), torch.empty_like(W)
        hs.haste_tail_step_sgd(desc, X, idx, W, None, pos, dY, None, opt, m, Wn, dX, 0, ws)
        return [dY.float(), m, dX]

    for call, op, n in zip((bwd_x, step, sgd), (hs.HASTE_OP_BWD_X, hs.HASTE_OP_TAIL_STEP, hs.HASTE_OP_TAIL_STEP_SGD), least):
        ref = call(hs.workspace(hs.haste_workspace_bytes(desc, op)))
        room = torch.full((n + 4096,), 0xa5, dtype=torch.uint8, device="cuda")
        got = call(room[:n])
        assert bool((room[n:] == 0xa5).all())
        for a, b in zip(got, ref):
            assert rel_err(a.cpu(), b.cpu()) < (1e-5 if f32 else SUM_TOL)
        with pytest.raises(Exception):
            call(room[:256])


@pytest.mark.parametrize("shape,dtype,least", SCRATCH)
def test_scratch_refusal(shape, dtype, least):
    """A tail step whose workspace is too small for one of its products launches none of them."""
    import torch
    import paper_2606_01117_amd as hs
    B, F_s, L, G, F_in = shape
    say("scratch refusal", shape, dtype)
    dt = torch.float32 if dtype == synth.DT_F32 else torch.bfloat16
    idx = torch.arange(F_in, dtype=torch.int32, device="cuda").repeat(L // G, 1)
    X, W = torch.ones((B, F_s), dtype=dt, device="cuda"), torch.ones((L, F_in), dtype=dt, device="cuda")
    m, dW, dX = (torch.full(s, 5.0, device="cuda") for s in ((L, F_in), (L, F_in), (B, F_s)))
    Wn, dY = torch.full((L, F_in), 5.0, dtype=dt, device="cuda"), torch.full((B, L), 5.0, dtype=dt, device="cuda")
    pos = torch.zeros((B, 1), dtype=torch.int32, device="cuda")
    desc = hs.make_desc(B, F_s, L, G, F_in, dtype)
    opt = hs.sgd_opts(0.1, 0.9, 1e-4)
    room = torch.empty(max(least), dtype=torch.uint8, device="cuda")
    step = lambda ws: hs.haste_tail_step(desc, X, idx, W, None, pos, dY, dW, None, 0, dX, 0, ws)
    sgd = lambda ws: hs.haste_tail_step_sgd(desc, X, idx, W, None, pos, dY, None, opt, m, Wn, dX, 0, ws)
    refused = 0
    for call, n in ((step, least[1]), (sgd, least[2])):
        for short in (256, least[0] // 256 * 256 // 8, least[0] // 256 * 256, n // 256 * 256 - 256, n):
            try:
                call(room[:n - short])
            except hs.HasteError as e:
                assert e.status == 3
                refused += 1
                for t in (m, dW, dX, Wn, dY):
                    assert bool((t == 5.0).all())
            else:                                 # a size that some kernels can do with
                for t in (m, dW, dX, Wn, dY):
                    t.fill_(5.0)
    assert refused >= 4
