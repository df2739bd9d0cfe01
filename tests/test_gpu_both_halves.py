"""Both halves of a layer in one launch (vcas_linear_backward on one stream): the bits of the two calls for the halves, at every
pair of tiles and on either side of the line up to which their tiles come to a CU each, with few and many samples kept."""
import numpy as np
import pytest
import torch

from workloads import BF16, F32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,N,T,K_in,K_out,rho,nu", [
    # bf16, dW in 64x64 tiles: a tile or two of each, ragged; contractions of one step and of many; beyond the line
    (BF16, 5, 37, 264, 136, 0.6, 0.5), (BF16, 1, 1, 8, 8, 1.0, 1.0), (BF16, 4, 33, 72, 8, 0.02, 0.02), (BF16, 16, 65, 520, 2056, 0.7, 0.6),
    (BF16, 9, 233, 776, 264, 1.0, 0.3), (BF16, 13, 300, 1032, 520, 1.0, 0.2), (BF16, 70, 60, 264, 264, 0.3, 0.3),
    (BF16, 10, 300, 520, 520, 0.5, 0.9),
    # bf16, dW in 128x128 tiles, either operand the narrower one; beyond the line
    (BF16, 3, 67, 1480, 1544, 0.7, 0.7), (BF16, 32, 40, 776, 3080, 0.5, 0.5), (BF16, 12, 50, 3080, 776, 0.4, 0.4), (BF16, 12, 300, 1480, 1544, 0.7, 0.2),
    # fp32: 64x64 and 64x64 tiles, 64x64 and 128x128, 128x128 and 64x64, 128x128 and 128x128; beyond the line
    (F32, 10, 100, 520, 520, 1.0, 1.0), (F32, 30, 64, 520, 2568, 0.5, 0.9), (F32, 20, 200, 776, 520, 0.5, 0.5),
    (F32, 20, 200, 776, 2200, 0.5, 0.5), (F32, 20, 200, 776, 3080, 1.0, 0.5), (F32, 8, 128, 768, 768, 0.5, 0.5),
    (F32, 20, 64, 520, 2568, 0.75, 0.5), (F32, 20, 200, 776, 2200, 0.5, 0.25),
], ids=lambda c: str(c))
def test_one_launch_is_the_two(dtype, N, T, K_in, K_out, rho, nu):
    from paper_2402_17227_amd import binding as vb
    from tests.gpu_util import plan_to_numpy
    vb.lib()
    real = torch.bfloat16 if dtype == BF16 else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(K_out)
    G = torch.randn((N * T, K_out), generator=gen, device="cuda")
    G = (G * torch.exp(torch.randn((N, 1), generator=gen, device="cuda")).repeat_interleave(T, 0)).to(real)
    X = torch.randn((N * T, K_in), generator=gen, device="cuda").to(real)
    W = (torch.randn((K_out, K_in), generator=gen, device="cuda") * 0.02).to(real)
    shape = vb.shape_of(N, T, K_in, K_out, dtype)
    ws = vb.make_workspace(shape)
    for draw in range(3):
        got = []
        for whole in (True, False):
            plan = vb.Plan.allocate(N, T)
            dX = torch.full((N * T, K_in), float("nan"), dtype=real, device="cuda")
            dW = torch.full((K_out, K_in), float("nan"), device="cuda")
            rng = vb.Rng(7, 2, draw)
            if whole:
                vb.vcas_linear_backward(shape, G, X, W, rho, nu, rng, True, plan, dX, dW, ws)
            else:
                vb.vcas_backward_data(shape, G, X, W, rho, rng, True, plan, dX, ws)
                vb.vcas_backward_weight(shape, G, X, rho, nu, rng, True, plan, dW, ws)
            got.append((plan_to_numpy(plan), dX, dW))
        (plan_a, dX_a, dW_a), (plan_b, dX_b, dW_b) = got
        for key in plan_a:
            assert np.array_equal(np.asarray(plan_a[key]), np.asarray(plan_b[key])), key
        bits = torch.int16 if dtype == BF16 else torch.int32
        assert torch.equal(dX_a.view(bits), dX_b.view(bits)) and torch.equal(dW_a.view(torch.int32), dW_b.view(torch.int32))
        assert bool(dX_a.isfinite().all()) and bool(dW_a.isfinite().all())


@pytest.mark.parametrize("dtype", [BF16, F32])
def test_the_timer_tells_the_halves_apart(dtype):
    """A layer that goes out in one launch: while the kernel timer is on either half is launched and counted, and the bits are the same."""
    from paper_2402_17227_amd import binding as vb
    N, T, K_in, K_out = 20, 200, 776, 520
    real = torch.bfloat16 if dtype == BF16 else torch.float32
    G, X, W = (torch.randn(size, device="cuda").to(real) for size in ((N * T, K_out), (N * T, K_in), (K_out, K_in)))
    shape = vb.shape_of(N, T, K_in, K_out, dtype)
    plan, ws = vb.Plan.allocate(N, T), vb.make_workspace(shape)
    got = []
    for timed in (False, True):
        dX, dW = torch.empty_like(X), torch.empty((K_out, K_in), device="cuda")
        if timed:
            vb.vcas_profile_begin()
        vb.vcas_linear_backward(shape, G, X, W, 0.5, 0.5, vb.Rng(7, 2, 0), True, plan, dX, dW, ws)
        if timed:
            (ms_x, n_x), (ms_w, n_w) = vb.vcas_profile_end()
            assert n_x == n_w == 1 and ms_x > 0.0 and ms_w > 0.0
        got.append((dX, dW))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


# fp32 sums that bf16 parts cannot hold (2^90) in single 32x32 blocks of dX and dW, which are formed again in plain fp32: beside
# them the blocks keep their bits whatever tile either way takes (dX 128x128 in one launch; apart 64x64, 64x128, 128x128)
@pytest.mark.parametrize("N,T,K_in,K_out", [(10, 100, 520, 520), (20, 200, 776, 520), (20, 200, 776, 2200), (30, 64, 520, 2568)])
def test_one_launch_is_the_two_beside_sums_formed_again(N, T, K_in, K_out):
    from paper_2402_17227_amd import binding as vb
    vb.lib()
    gen = torch.Generator(device="cuda").manual_seed(K_out)
    G = torch.randn((N * T, K_out), generator=gen, device="cuda")
    X = torch.randn((N * T, K_in), generator=gen, device="cuda")
    W = torch.randn((K_out, K_in), generator=gen, device="cuda") * 0.02
    rows = torch.arange(3, N, 5, device="cuda") * T + 37      # one token of one sample in five
    G[rows, 70] = 2.0 ** 50
    X[rows, 100] = 2.0 ** 40
    W[70, 65] = 2.0 ** 40
    shape = vb.shape_of(N, T, K_in, K_out, F32)
    ws = vb.make_workspace(shape)
    got = []
    for whole in (True, False):
        plan = vb.Plan.allocate(N, T)
        dX = torch.full((N * T, K_in), float("nan"), device="cuda")
        dW = torch.full((K_out, K_in), float("nan"), device="cuda")
        if whole:
            vb.vcas_linear_backward(shape, G, X, W, 0.5, 0.5, vb.Rng(7, 2, 0), True, plan, dX, dW, ws)
        else:
            vb.vcas_backward_data(shape, G, X, W, 0.5, vb.Rng(7, 2, 0), True, plan, dX, ws)
            vb.vcas_backward_weight(shape, G, X, 0.5, 0.5, vb.Rng(7, 2, 0), True, plan, dW, ws)
        got.append((dX, dW))
    (dX, dW), (dX_apart, dW_apart) = got
    assert torch.equal(dX, dX_apart) and torch.equal(dW, dW_apart)
    scale = (plan.maskA / plan.p.double()).nan_to_num(0.0).repeat_interleave(T)[:, None]
    kept = plan.idxW[:int(plan.cntW)].long()
    assert bool((kept[:, None] == rows[None]).any())
    G, X, W, Gw = G.double(), X.double(), W.double(), G[kept].double() * plan.scaleW[kept].double()[:, None]
    for out, want, terms in ((dX, G @ W * scale, G.abs() @ W.abs() * scale),
                             (dW, Gw.t() @ X[kept], Gw.abs().t() @ X[kept].abs())):
        assert float(out.abs().max()) > 2.0 ** 88
        # every element within fp32 sums of its own terms; 1e-12: dropped samples' rows are zero on both sides
        assert float(((out.double() - want).abs() / terms.clamp_min(1e-12)).max()) <= 2e-6
