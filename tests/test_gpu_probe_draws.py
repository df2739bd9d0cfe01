"""The variance probe over one draw, a chunk of eight, and more than one chunk, with both output tiles of the comparing
kernel, more samples than a workgroup has threads, rows beyond the one-workgroup samplers and rows so many that fewer draws go
together, against the oracle; and the plan it leaves: that of the last draw."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from workloads import BF16, F32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    (F32, 8, 24, 72, 64, 1), (BF16, 8, 24, 72, 64, 8), (F32, 5, 37, 264, 136, 9), (BF16, 5, 37, 264, 136, 17),
    (BF16, 3, 40, 776, 1032, 2), (F32, 3, 40, 776, 392, 2), (BF16, 1100, 2, 16, 24, 3), (F32, 7, 2400, 8, 8, 9),
    # rows whose vectors fill a chunk's scratch: seven draws together, then two, one after the other
    (F32, 70, 4700, 8, 8, 9), (BF16, 100, 10500, 8, 8, 3), (BF16, 1100, 2100, 8, 8, 3),
], ids=lambda c: "x".join(map(str, c)))
def test_probe_over_chunks_of_draws(case):
    from paper_2402_17227_amd import binding as vb
    from tests.gpu_util import compare_plan, plan_to_numpy, to_device
    dtype, N, T, K_in, K_out, M = case
    sp = workloads.LayerSpec("probe", dtype, N, T, K_in, K_out, 0.5, 0.5, layer=4, seed=5, gen_seed=M, token_sigma=0.5)
    G, X, _ = workloads.make_layer(sp)
    shape = vb.shape_of(N, T, K_in, K_out, dtype)
    plan, ws = vb.Plan.allocate(N, T), vb.make_workspace(shape)
    out = torch.full((4,), float("nan"), dtype=torch.float64, device="cuda")
    vb.vcas_variance_probe(shape, to_device(G, dtype), to_device(X, dtype), 0.5, 0.5, vb.Rng(5, 4, 10), M, plan, out, ws)
    torch.cuda.synchronize()
    want = oracle.variance_probe(G, X, dtype, N, T, 0.5, 0.5, 5, 4, 10, M)
    got = out.cpu().numpy()
    # closed forms: the same fp32 inputs, fp64 sums; squared differences of dW: the rounding of dW (fp32 sums; in bf16 also
    # of its scaled operand, 2^-9) against differences that are sampling noise, of the size of dW itself
    np.testing.assert_allclose(got[:2], want[:2], rtol=1e-9)
    np.testing.assert_allclose(got[2:], want[2:], rtol=1e-4 if dtype == F32 else 3e-2)
    compare_plan(plan_to_numpy(plan), oracle.sampling_plan(G, X, dtype, N, T, 0.5, 0.5, 5, 4, 10 + M - 1))


# Where nothing is left to chance a draw is the exact gradient and its distance is zero, whichever kernels form the two: bf16
# exact gradients of many rows (packed, in slices) and of few, fp32 in slices, products beyond the comparing kernel (K_in
# K_out of 2^28 and more; one draw after the other), more than one chunk of draws
@pytest.mark.parametrize("case", [
    (BF16, 8, 300, 264, 136, 9), (BF16, 3, 40, 776, 1032, 2), (F32, 8, 300, 264, 136, 3), (F32, 5, 37, 72, 64, 9),
    (F32, 2, 6, 16392, 16392, 2),
], ids=lambda c: "x".join(map(str, c)))
def test_probe_without_a_choice(case):
    from paper_2402_17227_amd import binding as vb
    dtype, N, T, K_in, K_out, M = case
    gen = torch.Generator(device="cuda").manual_seed(M)
    real = torch.bfloat16 if dtype == BF16 else torch.float32
    G = torch.randn((N * T, K_out), generator=gen, device="cuda").to(real)
    X = torch.randn((N * T, K_in), generator=gen, device="cuda").to(real)
    shape = vb.shape_of(N, T, K_in, K_out, dtype)
    plan, ws = vb.Plan.allocate(N, T), vb.make_workspace(shape)

    def probe(rho, nu):
        out = torch.full((4,), float("nan"), dtype=torch.float64, device="cuda")
        vb.vcas_variance_probe(shape, G, X, rho, nu, vb.Rng(5, 4, 10), M, plan, out, ws)
        return out.tolist()

    assert probe(1.0, 1.0) == [0.0] * 4
    only_tokens = probe(1.0, 0.5)
    assert only_tokens[0] == only_tokens[2] == 0.0 and only_tokens[1] > 0.0 and only_tokens[3] > 0.0
    # half of the budget is enough for every sample that is not zero, and a zero row is not one more choice
    G[(N // 2) * T:] = 0
    X[1] = 0
    assert probe(0.5, 1.0) == [0.0] * 4
    assert probe(0.25, 1.0)[2] > 0.0


# Products of which some sums (2^90) are beyond what the bf16 parts of fp32 values hold and are formed again, in the comparing
# kernel's 64x64 and 128x128 tiles
@pytest.mark.parametrize("K_in,K_out,M", [(264, 136, 2), (776, 392, 2), (776, 776, 2)])
def test_probe_of_sums_beyond_the_parts(K_in, K_out, M):
    from paper_2402_17227_amd import binding as vb
    from tests.gpu_util import to_device
    N, T = 6, 40
    sp = workloads.LayerSpec("probe", F32, N, T, K_in, K_out, 0.5, 0.5, layer=4, seed=5, gen_seed=M, token_sigma=0.5)
    G, X, _ = workloads.make_layer(sp)
    G[::3, 70] *= np.float32(2.0 ** 50)      # tokens of every sample, so that either mask has a choice
    X[::3, 100] *= np.float32(2.0 ** 40)
    shape = vb.shape_of(N, T, K_in, K_out, F32)
    plan, ws = vb.Plan.allocate(N, T), vb.make_workspace(shape)
    out = torch.full((4,), float("nan"), dtype=torch.float64, device="cuda")
    vb.vcas_variance_probe(shape, to_device(G, F32), to_device(X, F32), 0.5, 0.2, vb.Rng(5, 4, 10), M, plan, out, ws)
    want = oracle.variance_probe(G, X, F32, N, T, 0.5, 0.2, 5, 4, 10, M)
    got = out.cpu().numpy()
    assert want[2:].min() > 2.0 ** 150
    np.testing.assert_allclose(got[:2], want[:2], rtol=1e-9)
    np.testing.assert_allclose(got[2:], want[2:], rtol=1e-4)
