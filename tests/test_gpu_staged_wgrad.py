"""The bf16 weight gradient whose operands are scaled on their way to LDS: 64x64 tiles with two wavefronts to a block and 128x128
tiles, whole and in slices of which all, some, one or none have tokens, either operand the scaled one, ragged columns and last steps,
against 64 bits on the rounded operand."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,K_in,K_out,kept", [
    # 64x64, whole
    (2100, 768, 768, 2100), (2100, 776, 712, 65), (2100, 712, 776, 64), (2100, 768, 768, 1), (2100, 768, 768, 0), (50, 8, 8, 50), (1, 72, 200, 1),
    # 64x64 in eight slices
    (8000, 256, 264, 8000), (8000, 264, 256, 1025), (8000, 264, 256, 1023), (8000, 256, 264, 257), (8000, 256, 264, 129), (8000, 256, 264, 127),
    (8000, 256, 264, 0),
    # 128x128, whole and in slices
    (1500, 776, 3080, 1500), (1500, 3080, 776, 191), (1500, 3080, 776, 1), (4001, 776, 768, 4001), (4001, 768, 776, 700), (4001, 768, 776, 129),
    (4001, 768, 776, 2)])
def test_scaled_on_the_way(R, K_in, K_out, kept):
    from paper_2402_17227_amd import binding as vb
    vb.lib()
    gen = torch.Generator(device="cuda").manual_seed(R + kept)
    G = torch.randn((R, K_out), generator=gen, device="cuda").bfloat16()
    X = torch.randn((R, K_in), generator=gen, device="cuda").bfloat16()
    scale = torch.rand(R, generator=gen, device="cuda") * 3 + 1
    rows = torch.randperm(R, generator=gen, device="cuda")[:kept].sort().values
    on = torch.zeros(R, dtype=torch.bool, device="cuda")
    on[rows] = True
    G[~on], X[~on] = float("nan"), float("inf")    # tokens that are not kept are not read
    idx = torch.full((R,), -1, dtype=torch.int32, device="cuda")
    idx[:kept] = rows.int()
    cnt = torch.tensor([kept], dtype=torch.int32, device="cuda")
    shape = vb.shape_of(1, R, K_in, K_out, vb.VCAS_BF16)
    dW = torch.full((K_out, K_in), float("nan"), device="cuda")
    vb.vcas_sampled_wgrad(shape, G, X, scale, idx, cnt, dW, vb.make_workspace(shape))
    g, x = G[rows].float(), X[rows].float()
    if K_out < K_in:     # the narrower operand is scaled, and rounded once
        g = (g * scale[rows, None]).bfloat16().float()
    else:
        x = (x * scale[rows, None]).bfloat16().float()
    want = g.double().t() @ x.double()
    if not kept:
        assert float(dW.abs().sum()) == 0.0
        return
    off = dW.double() - want
    # products of two bf16 values are exact; sums rounded once per 16 terms and per slice
    bound = (math.sqrt(kept / 16) + 4) * 2.0 ** -24
    assert float(off.norm() / want.norm()) <= bound
    for dim in (0, 1):
        assert float((off.norm(dim=dim) / want.norm(dim=dim)).max()) <= 4 * bound   # a row has its own spread


@pytest.mark.parametrize("packed,N,T,widths", [
    # either side of the line at 1300 expected tokens, of tiles of 128x128 and 64x64; few tokens, mixtures that end one launch and start the next
    (False, 2, 650, ((768, 776), (72, 200))), (True, 2, 651, ((768, 776), (72, 200))), (False, 3, 5, ((512, 512), (520, 384), (8, 8))),
    (False, 4, 64, ((512, 1032), (64, 64), (1032, 512), (504, 512))),
    # either side of 640 tiles of 128x128; one wide layer packs all of its group (two layers; the third is the next group)
    (False, 2, 100, ((2056, 4600),)), (True, 2, 100, ((2056, 4872),)), ((True, True, False), 1, 300, ((264, 136), (2056, 4872), (520, 520))),
    # packed, ragged columns and last steps: 64x64 tiles (fewer than sixteen of 128x128 in the launch), 128x128 in slices, 256x256 (64 of
    # them and more), either operand the packed one
    (True, 2, 1025, ((264, 136),)), (True, 3, 700, ((8, 8), (136, 264))), (True, 2, 1025, ((768, 776), (72, 200))), (True, 4, 513, ((768, 776), (72, 200))),
    (True, 1, 2333, ((1544, 3080), (2056, 2120))), (True, 3, 777, ((3080, 1544), (2120, 2056)))])
def test_beside_the_dgrads_of_a_stack(packed, N, T, widths):
    """Entries of a stack with wgrad_fill 64: dW of every layer against 64 bits on what its plan kept, and the form they take."""
    from tests.gpu_util import packs_the_kept_rows
    from paper_2402_17227_amd import binding as vb
    vb.lib()
    gen = torch.Generator(device="cuda").manual_seed(N * T)
    R = N * T
    entries, without, keep = [], [], []
    for l, (K_in, K_out) in enumerate(widths):
        shape = vb.shape_of(N, T, K_in, K_out, vb.VCAS_BF16)
        G = torch.randn((R, K_out), generator=gen, device="cuda").bfloat16()
        X = torch.randn((R, K_in), generator=gen, device="cuda").bfloat16()
        W = torch.randn((K_out, K_in), generator=gen, device="cuda").bfloat16()
        plan, ws = vb.Plan.allocate(N, T), vb.make_workspace(shape)
        dX, dW = torch.empty_like(X), torch.full((K_out, K_in), float("nan"), device="cuda")
        for some, out in ((entries, dW), (without, None)):
            some.append(vb.layer_args(shape, G, X, W, 1.0, 0.999, vb.Rng(2, l, 0), True, plan, dX, out, ws, wgrad_fill=64))
        keep.append((G, X, W, plan, ws, dX, dW))
    streams = torch.cuda.Stream(), torch.cuda.Stream()
    stack, plans = vb.make_stack(entries), vb.make_stack(without)
    call = lambda stack: vb.vcas_backward_stack(stack, len(entries), *streams)
    for l, (G, X, W, plan, ws, dX, dW) in enumerate(keep):
        assert packs_the_kept_rows(ws, lambda: call(stack), lambda: call(plans)) == (packed if isinstance(packed, bool) else packed[l]), l
        cnt = int(plan.cntW)
        rows = plan.idxW[:cnt].long()
        scale = plan.scaleW[rows]
        g, x = G[rows].float(), X[rows].float()
        if G.shape[1] < X.shape[1]:
            g = (g * scale[:, None]).bfloat16().float()
        else:
            x = (x * scale[:, None]).bfloat16().float()
        want = g.double().t() @ x.double()
        assert float((dW.double() - want).norm() / want.norm()) <= (math.sqrt(cnt / 16) + 4) * 2.0 ** -24
