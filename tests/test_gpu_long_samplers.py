"""SampleW on both sides of the lines between its forms: one element per thread up to sixteen in one workgroup, the three
launches for more rows than that (scores in 32 or 64 registers per thread, or read again every round), the list from the
mask bytes or from counts, more samples than a workgroup has threads.  Plans bit for bit against the oracle."""
import pytest
import torch

import oracle
import workloads
from workloads import BF16, F32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vb():
    from paper_2402_17227_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


CASES = [  # dtype, N, T, K_in, K_out, rho, nu
    (BF16, 1, 1024, 8, 8, 1.0, 0.5), (BF16, 5, 205, 8, 16, 0.8, 0.5), (F32, 4, 2048, 8, 8, 0.5, 0.3),
    (BF16, 33, 249, 16, 8, 0.7, 0.4), (BF16, 16, 1024, 8, 8, 0.5, 0.5),
    (BF16, 113, 145, 8, 8, 0.7, 0.4),            # 16385 rows
    (F32, 32, 1024, 8, 8, 0.6, 0.2), (BF16, 3, 10923, 8, 8, 1.0, 0.5),
    (BF16, 64, 1024, 8, 8, 0.5, 0.5), (F32, 2048, 31, 8, 8, 0.5, 0.05),
    (BF16, 3, 21846, 8, 8, 0.7, 0.6),            # 65538 rows
    (BF16, 40, 13, 520, 8, 0.5, 0.02),           # sums in which almost nothing is kept
    (F32, 64, 2048, 8, 8, 0.6, 0.5), (BF16, 11, 11916, 8, 8, 0.7, 0.4),    # 131072 rows, 131076
    (F32, 1111, 500, 8, 8, 0.5, 0.3),            # more counts than a workgroup has threads
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("token_sampling", [True, False])
def test_plan_of_long_vectors(vb, case, token_sampling):
    from tests.gpu_util import compare_plan, rel_l2, run_layer_gpu
    dtype, N, T, K_in, K_out, rho, nu = case
    sp = workloads.LayerSpec("long", dtype, N, T, K_in, K_out, rho, nu, layer=2, seed=9, gen_seed=T, sample_sigma=1.5,
                             token_sigma=0.5)
    G, X, W = workloads.make_layer(sp)
    want, want_dX, want_dW = oracle.linear_backward(G, X, W, dtype, N, T, rho, nu, sp.seed, sp.layer, 0,
                                                    token_sampling=token_sampling)
    plan, dX, dW = run_layer_gpu(sp, G, X, W, token_sampling=token_sampling)
    compare_plan(plan, want)
    tol = 1e-2 if dtype == BF16 else 1e-5
    assert rel_l2(dX, want_dX) <= tol and rel_l2(dW, want_dW) <= tol


@pytest.mark.parametrize("R", [512, 20000])
def test_siblings_with_long_vectors(vb, R):
    """V, K and Q in one stack launch against calls of their own."""
    N, T, K = 20, R // 20, 64
    s2, s3 = torch.cuda.Stream(), torch.cuda.Stream()
    outs = []
    for how in ("stack", "alone"):
        entries, keep = [], []
        for l in range(3):
            sp = workloads.LayerSpec("sib", BF16, N, T, K, K, 0.6, 0.5, layer=l, seed=4, gen_seed=l)
            g, x, w = (vb.to_device(a, BF16) for a in workloads.make_layer(sp))
            shape, plan = vb.shape_of(N, T, K, K, BF16), vb.Plan.allocate(N, T)
            ws = vb.make_workspace(shape)
            dX = torch.zeros((N * T, K), dtype=torch.bfloat16, device="cuda")
            dW = torch.zeros((K, K), device="cuda")
            rng = vb.Rng(sp.seed, sp.layer, 0)
            if how == "alone":
                vb.vcas_linear_backward(shape, g, x, w, 0.6, 0.5, rng, True, plan, dX, dW, ws)
            entries.append(vb.layer_args(shape, g, x, w, 0.6, 0.5, rng, True, plan, dX, dW, ws, sibling=l > 0))
            keep.append((g, x, w, plan, ws, dX, dW))
        if how == "stack":
            vb.vcas_backward_stack(vb.make_stack(entries), 3, s2, s3)
        torch.cuda.synchronize()
        outs.append(keep)
    for a, b in zip(*outs):
        n = int(a[3].cntW.item())
        assert n == int(b[3].cntW.item()) and torch.equal(a[3].idxW[:n], b[3].idxW[:n])
        assert torch.equal(a[3].q.view(torch.int32), b[3].q.view(torch.int32)) and torch.equal(a[3].scaleW, b[3].scaleW)
        assert torch.equal(a[5], b[5]) and torch.equal(a[6], b[6])


def test_plans_of_many_rows_take_linear_time(vb):
    """Four times the rows, in the launches behind the keep rule (norms given, no token sampling, no dW): about four times
    the time, where work that grows with the square of the rows would take sixteen times."""
    took = []
    for R in (1 << 23, 1 << 25):
        shape = vb.shape_of(64, R // 64, 8, 8, F32)
        G, xsq = torch.randn((R, 8), device="cuda"), torch.rand(R, device="cuda")
        plan, ws = vb.Plan.allocate(64, R // 64), vb.make_workspace(shape)
        vb.vcas_backward_data(shape, G, G, None, 0.7, vb.Rng(1, 2, 0), False, plan, None, ws)
        best = float("inf")
        for _ in range(4):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            vb.vcas_backward_weight_cached(shape, G, G, xsq, 0.7, 0.5, vb.Rng(1, 2, 0), False, plan, None, ws)
            end.record()
            torch.cuda.synchronize()
            best = min(best, begin.elapsed_time(end))
        took.append(best)
        kept = plan.maskA.bool().repeat_interleave(R // 64).nonzero()[:, 0]
        assert torch.equal(plan.idxW[:kept.numel()].long(), kept) and int(plan.cntW.item()) == kept.numel()
    assert took[1] <= 8 * took[0], took
