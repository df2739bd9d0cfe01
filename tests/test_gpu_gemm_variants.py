"""One case on each side of every line at which a launch picks another GEMM kernel, at sizes where that kernel can go
wrong (ragged edges of its tiles, contraction remainders, a single step, nothing kept): the whole path against the
oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from workloads import BF16, F32

pytestmark = pytest.mark.gpu
TOL = {F32: 1e-5, BF16: 1e-2}


@pytest.fixture(scope="module")
def vb():
    from paper_2402_17227_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


F32_CASES = [
    # dgrad with 32x32 tiles (at most 256 of them), eight wavefronts per tile; wgrad with 32x32 tiles in slices
    (3, 11, 8, 8, 0.5, 0.5), (3, 33, 264, 72, 0.7, 0.6), (7, 40, 96, 520, 0.6, 0.5), (40, 64, 64, 136, 1.0, 1.0),
    # dgrad with 32x64 tiles
    (5, 131, 552, 200, 1.0, 0.3),
    # 264 tiles of 64x64, so 64x128 (those and the other tiles from bf16 parts: test_fp32_dgrad_tiles)
    (9, 233, 456, 72, 1.0, 0.5),
    # wgrad with 128x128 tiles from bf16 parts: full, remainder and single steps of 32 tokens, nothing kept
    (4, 47, 1608, 1928, 0.5, 0.5), (2, 16, 1608, 1928, 1.0, 1.0), (2, 5, 1608, 1928, 0.02, 0.02),
]


@pytest.mark.parametrize("case", F32_CASES, ids=lambda c: "x".join(map(str, c)))
def test_fp32_kernels_at_their_edges(vb, case):
    _against_oracle(F32, *case)


BF16_CASES = [
    # wgrad gathering with 64x64 tiles: fewer than 32 of them, 256, ragged; G scaled, X scaled
    (3, 11, 8, 8, 0.5, 0.5), (9, 233, 264, 136, 0.6, 0.7), (9, 233, 136, 264, 0.7, 0.7), (8, 256, 1024, 1024, 1.0, 0.99),
    # nothing kept, one token; whole and in slices
    (2, 5, 72, 200, 0.02, 0.02), (1, 1, 72, 200, 1.0, 1.0), (1, 1000, 64, 72, 1.0, 1.0), (1, 1025, 64, 72, 1.0, 1.0),
    # 18 x 19 tiles, ragged, either side scaled; 128x128 tiles, ragged, either side scaled
    (3, 67, 1096, 1160, 0.7, 0.7), (3, 67, 1160, 1096, 0.7, 0.7), (8, 257, 1096, 1160, 1.0, 0.9),
    (3, 67, 1480, 1544, 0.7, 0.7), (3, 67, 1544, 1480, 0.7, 0.7), (1, 129, 1480, 1544, 1.0, 1.0), (1, 321, 1480, 1544, 1.0, 1.0),
    # gathering over whole, partial and single steps of 64 tokens, with 64x64 tiles; 17 x 17 tiles of 128x128
    (1, 64, 264, 264, 1.0, 1.0), (1, 65, 264, 264, 1.0, 1.0), (1, 200, 264, 264, 1.0, 1.0), (1, 257, 264, 264, 1.0, 1.0),
    (1, 513, 264, 264, 1.0, 1.0), (1, 129, 1096, 1160, 1.0, 1.0), (1, 321, 1096, 1160, 1.0, 1.0), (3, 67, 2056, 2120, 0.7, 0.7),
    # 128x128 tiles of wide matrices
    (1, 300, 3592, 3688, 1.0, 1.0), (2, 200, 3688, 3592, 1.0, 0.8), (2, 300, 3464, 3208, 1.0, 0.9), (2, 300, 3848, 4104, 1.0, 0.9),
]


@pytest.mark.parametrize("case", BF16_CASES, ids=lambda c: "x".join(map(str, c)))
def test_bf16_kernels_at_their_edges(vb, case):
    _against_oracle(BF16, *case)


# The packed form of a layer on its own, ragged in columns and tokens, either side the packed one: 128x128 tiles in slices; 256x256
# tiles, 15 x 15 of them (one for nearly every CU); below 192 and beyond 256 of those (14 x 13, 16 x 17) 128x128 tiles again
@pytest.mark.parametrize("case", [
    (1, 4101, 1304, 1496, 1.0, 1.0), (3, 1501, 1496, 1304, 1.0, 0.93), (1, 877, 3592, 3688, 1.0, 1.0), (2, 501, 3688, 3592, 1.0, 0.9),
    (1, 2501, 3464, 3208, 1.0, 1.0), (2, 907, 3848, 4104, 1.0, 0.97)], ids=lambda c: "x".join(map(str, c)))
def test_packed_weight_gradients_at_their_edges(vb, case):
    from tests.gpu_util import packs_the_kept_rows
    _against_oracle(BF16, *case)
    N, T, K_in, K_out, rho, nu = case
    shape = vb.shape_of(N, T, K_in, K_out, BF16)
    G, X = (torch.randn((N * T, K), device="cuda").bfloat16() for K in (K_out, K_in))
    plan, ws, dW = vb.Plan.allocate(N, T), vb.make_workspace(shape), torch.empty((K_out, K_in), device="cuda")
    call = lambda out: vb.vcas_linear_backward(shape, G, X, None, rho, nu, vb.Rng(3, 1, 0), True, plan, None, out, ws)
    assert packs_the_kept_rows(ws, lambda: call(dW), lambda: call(None))


def _against_oracle(dtype, N, T, K_in, K_out, rho, nu):
    from tests.gpu_util import compare_plan, rel_l2, rel_l2_rows, rel_l2_tiles, run_layer_gpu
    sp = workloads.LayerSpec("edge", dtype, N, T, K_in, K_out, rho, nu, layer=5, seed=31, gen_seed=N + T, token_sigma=0.5)
    G, X, W = workloads.make_layer(sp)
    want, want_dX, want_dW = oracle.linear_backward(G, X, W, dtype, N, T, rho, nu, sp.seed, sp.layer, 0)
    plan, dX, dW = run_layer_gpu(sp, G, X, W)
    compare_plan(plan, want)
    assert rel_l2(dX, want_dX) <= TOL[dtype] and rel_l2(dW, want_dW) <= TOL[dtype]
    assert rel_l2_rows(dX, want_dX) <= 2 * TOL[dtype] and rel_l2_tiles(dW, want_dW) <= 2 * TOL[dtype]


@pytest.mark.parametrize("T,K_in,jacobian", [(4096, 8, False), (4099, 200, True)])
def test_fp32_tensors_beyond_32_bit_offsets(vb, T, K_in, jacobian):
    """G of more than 2 GiB: rows at both ends of it against a product in double precision; one column tile, and four, the last one
    ragged, with tiles of rows that straddle two samples and a Jacobian."""
    N, K_out = 16, 8200
    R = N * T
    shape = vb.shape_of(N, T, K_in, K_out, vb.VCAS_F32)
    gen = torch.Generator(device="cuda").manual_seed(1)
    G = torch.randn((R, K_out), generator=gen, device="cuda")
    X = torch.randn((R, K_in), generator=gen, device="cuda")
    W = torch.randn((K_out, K_in), generator=gen, device="cuda") * 0.02
    p = torch.full((N,), 0.5, device="cuda")
    idxA = torch.tensor([0, N - 1] + [0] * (N - 2), dtype=torch.int32, device="cuda")
    cntA = torch.tensor([2], dtype=torch.int32, device="cuda")
    dX = torch.full((R, K_in), float("nan"), device="cuda")
    kept = torch.cat([torch.arange(T, device="cuda"), torch.arange(R - T, R, device="cuda")])
    want = 2.0 * (G[kept].double() @ W.double())
    if jacobian:
        J = torch.rand((R, K_in), generator=gen, device="cuda")
        vb.vcas_sampled_dgrad_jac(shape, G, W, p, idxA, cntA, J, dX)
        want *= J[kept].double()
    else:
        vb.vcas_sampled_dgrad(shape, G, W, p, idxA, cntA, dX)
    off = dX[kept].double() - want
    # sums of 8200 fp32 products: sqrt(8200) 2^-24 = 5e-6, a row or a column alike
    assert float((off.norm(dim=1) / want.norm(dim=1)).max()) <= 3e-5 and float((off.norm(dim=0) / want.norm(dim=0)).max()) <= 1e-5
    assert float(off.norm() / want.norm()) <= 1e-5
    assert float(dX[T:R - T].abs().max()) == 0.0
    tokens = torch.cat([kept[:200], kept[-57:]]).to(torch.int32)
    idxW = torch.zeros(R, dtype=torch.int32, device="cuda")
    idxW[:tokens.numel()] = tokens
    cntW = torch.tensor([tokens.numel()], dtype=torch.int32, device="cuda")
    scale = torch.rand(R, generator=gen, device="cuda") + 1.0
    dW = torch.full((K_out, K_in), float("nan"), device="cuda")
    ws = vb.make_workspace(shape)
    vb.vcas_sampled_wgrad(shape, G, X, scale, idxW, cntW, dW, ws)
    t = tokens.long()
    want = (G[t].double() * scale[t].double()[:, None]).t() @ X[t].double()
    assert float((dW.double() - want).norm() / want.norm()) <= 1e-5


# 256x256 tiles of dgrad with the last round's tiles cut into quarters: whole tiles and quarters (287 = 256 + 31 tiles,
# 256 + 24), quarters only (28 and 63 tiles: one to a workgroup; 126: two), none kept, too many for quarters (196), a
# contraction too short for them; ragged in rows, columns and contraction
@pytest.mark.parametrize("K_out,kept", [(1544, 40), (1544, 39), (1544, 3), (1544, 8), (1544, 17),
                                        (1544, 0), (1544, 27), (1536, 40), (1528, 40)])
def test_dgrad_last_round_in_quarters(vb, K_out, kept):
    N, T, K_in = 40, 257, 1608
    R = N * T
    shape = vb.shape_of(N, T, K_in, K_out, vb.VCAS_BF16)
    gen = torch.Generator(device="cuda").manual_seed(K_out + kept)
    G = torch.randn((R, K_out), generator=gen, device="cuda").bfloat16()
    W = (torch.randn((K_out, K_in), generator=gen, device="cuda") * 0.02).bfloat16()
    J = torch.rand((R, K_in), generator=gen, device="cuda").bfloat16()
    p = torch.rand(N, generator=gen, device="cuda") * 0.5 + 0.5
    chosen = torch.randperm(N, generator=gen, device="cuda")[:kept].sort().values
    idxA = torch.zeros(N, dtype=torch.int32, device="cuda")
    idxA[:kept] = chosen.int()
    cntA = torch.tensor([kept], dtype=torch.int32, device="cuda")
    dX = torch.full((R, K_in), float("nan"), dtype=torch.bfloat16, device="cuda")
    blocks = torch.zeros(vb.vcas_sq_blocks_bytes(R, K_in) // 4, device="cuda")
    vb.vcas_sampled_dgrad_norms(shape, G, W, p, idxA, cntA, J, dX, blocks)
    mask = torch.zeros(N, device="cuda")
    mask[chosen] = 1.0 / p[chosen]
    want = (G.double() @ W.double()) * mask.double().repeat_interleave(T)[:, None] * J.double()
    got = dX.double()
    assert bool(torch.isfinite(got).all())
    dropped = mask.repeat_interleave(T) == 0
    assert float(got[dropped].abs().sum()) == 0.0
    if kept:
        # fp32 sums rounded once to bf16: 2^-9 / sqrt(3) = 1.1e-3; a row or a 64-column block alike
        off = (got - want)[~dropped]
        assert float((off.norm(dim=1) / want[~dropped].norm(dim=1)).max()) <= 5e-3
        assert float((off.norm(dim=0) / want[~dropped].norm(dim=0)).max()) <= 5e-3
        rows = blocks.view(-1, R, 4).permute(1, 0, 2).reshape(R, -1)[:, :(K_in + 63) // 64].double().sum(1)
        assert float(((rows - (got * got).sum(1)).abs() / (got * got).sum(1).clamp_min(1e-30))[~dropped].max()) <= 1e-5


# On both sides of the lines between the forms of a weight gradient: 64x64 tiles whole and in slices (16 and 64 of them), in two
# slices and 128x128 tiles in five (768x768), 64x64 and 128x128 tiles whole, 128x128 tiles and the packed form, with and without slices
@pytest.mark.parametrize("K_in,K_out,tokens,packed", [
    (256, 256, 1096, False), (256, 256, 1104, False), (512, 512, 1424, False), (512, 512, 1432, False), (768, 768, 3096, False),
    (768, 768, 3104, False), (1304, 1496, 728, False), (1304, 1496, 736, False), (1304, 1496, 3960, False), (1304, 1496, 3968, True),
    (1096, 1032, 7392, False), (1096, 1032, 7400, True), (776, 3080, 5392, False), (776, 3080, 5400, True), (3400, 3456, 968, False),
    (3400, 3456, 976, True)])
def test_form_of_a_small_weight_gradient(vb, K_in, K_out, tokens, packed):
    from tests.gpu_util import packs_the_kept_rows
    N, T = 8, tokens // 8
    shape = vb.shape_of(N, T, K_in, K_out, vb.VCAS_BF16)
    gen = torch.Generator(device="cuda").manual_seed(tokens)
    G = torch.randn((tokens, K_out), generator=gen, device="cuda").bfloat16()
    X = torch.randn((tokens, K_in), generator=gen, device="cuda").bfloat16()
    plan, ws = vb.Plan.allocate(N, T), vb.make_workspace(shape)
    dW = torch.full((K_out, K_in), float("nan"), device="cuda")
    call = lambda out: vb.vcas_linear_backward(shape, G, X, None, 1.0, 1.0, vb.Rng(3, 1, 0), True, plan, None, out, ws)
    assert packs_the_kept_rows(ws, lambda: call(dW), lambda: call(None)) == packed
    want = G.double().t() @ X.double()
    # fp32 sums of exact products, in any order: sqrt(7400) 2^-24 = 5e-6
    assert float((dW.double() - want).norm() / want.norm()) <= 1e-5
    # vcas_sampled_wgrad, which knows no expected count, takes all rows for kept: here that is so
    other = torch.full((K_out, K_in), float("nan"), device="cuda")
    vb.vcas_sampled_wgrad(shape, G, X, plan.scaleW, plan.idxW, plan.cntW, other, ws)
    assert torch.equal(dW, other)


def test_gathering_layers_of_a_stack_share_launches(vb):
    """Twenty siblings that gather (sixteen to a launch), one in the middle without a dW and one of more than 1300 expected tokens
    that takes the packed form: three gathering launches around one packed launch, each dW the bits of a call of its own."""
    from tests.gpu_util import packs_the_kept_rows
    N, T, K = 8, 32, 128
    gen = torch.Generator(device="cuda").manual_seed(6)
    one = lambda *size: torch.randn(size, generator=gen, device="cuda").bfloat16()
    entries, keep = [], []
    for l in range(22):
        tokens, ratios = (8 * T, (0.9, 0.9)) if l == 4 else (T, (0.7, 0.5))
        shape = vb.shape_of(N, tokens, K, K, vb.VCAS_BF16)
        G, X, W = one(N * tokens, K), one(N * tokens, K), one(K, K)
        plan, ws = vb.Plan.allocate(N, tokens), vb.make_workspace(shape)
        dX, dW = torch.empty_like(X), torch.full((K, K), float("nan"), device="cuda")
        entries.append(vb.layer_args(shape, G, X, W, *ratios, vb.Rng(2, l, 0), True, plan, dX, None if l == 2 else dW, ws,
                                     sibling=l > 0, wgrad_fill=64 if l == 4 else 0))
        keep.append((shape, ratios, G, X, W, plan, ws, dX, dW))
    streams = torch.cuda.Stream(), torch.cuda.Stream()
    shape, ratios, G, X, W, plan, ws, dX, dW = keep[4]
    alone = lambda dW: vb.vcas_backward_stack(vb.make_stack([vb.layer_args(
        shape, G, X, W, *ratios, vb.Rng(2, 4, 0), True, plan, dX, dW, ws, wgrad_fill=64)]), 1, *streams)
    assert packs_the_kept_rows(ws, lambda: alone(dW), lambda: alone(None))
    dW.fill_(float("nan"))
    stack = vb.make_stack(entries)
    vb.vcas_profile_begin()
    vb.vcas_backward_stack(stack, 22, *streams)
    torch.cuda.synchronize()
    assert vb.vcas_profile_end()[1][1] == 4
    for l, (shape, ratios, G, X, W, plan, ws, dX, dW) in enumerate(keep):
        if l in (2, 4):
            assert bool(torch.isnan(dW).any()) == (l == 2)
            continue
        want = torch.full((K, K), float("nan"), device="cuda")
        vb.vcas_linear_backward(shape, G, X, W, *ratios, vb.Rng(2, l, 0), True, plan, dX, want, ws)
        assert torch.equal(dW.view(torch.int32), want.view(torch.int32)), l


def test_layers_of_one_big_tile_per_cu_in_a_stack(vb):
    """Two layers of 14 x 14 tiles of 256x256 and one of 13 x 14 in a stack with wgrad_fill 0: the bits of calls of their
    own, all of them packed."""
    from tests.gpu_util import packs_the_kept_rows
    N, T = 2, 1301
    entries, keep = [], []
    gen = torch.Generator(device="cuda").manual_seed(8)
    one = lambda *size: torch.randn(size, generator=gen, device="cuda").bfloat16()
    for l, (K_in, K_out) in enumerate([(3400, 3456), (3400, 3456), (3400, 3208)]):
        shape = vb.shape_of(N, T, K_in, K_out, vb.VCAS_BF16)
        G, X = one(N * T, K_out), one(N * T, K_in)
        plan, ws = vb.Plan.allocate(N, T), vb.make_workspace(shape)
        dW = torch.full((K_out, K_in), float("nan"), device="cuda")
        entries.append(vb.layer_args(shape, G, X, None, 1.0, 1.0, vb.Rng(2, l, 0), True, plan, None, dW, ws))
        keep.append((shape, G, X, plan, ws, dW))
    vb.vcas_backward_stack(vb.make_stack(entries), 3, *[torch.cuda.Stream() for _ in range(2)])
    torch.cuda.synchronize()
    for l, (shape, G, X, plan, ws, dW) in enumerate(keep):
        want = torch.full_like(dW, float("nan"))
        call = lambda out: vb.vcas_linear_backward(shape, G, X, None, 1.0, 1.0, vb.Rng(2, l, 0), True, plan, None, out, ws)
        assert packs_the_kept_rows(ws, lambda: call(want), lambda: call(None))
        assert torch.equal(dW.view(torch.int32), want.view(torch.int32)), l


# fp32 dgrad from bf16 parts: 64x64 tiles (8 x 31 of them), with contractions of less than, exactly and just beyond a step of 64;
# 64x128 tiles up to 256 of them, and for contractions of up to 128 beyond; 128x128 tiles, with steps of 32 that are full, half and single;
# samples dropped, Jacobians, rows and columns ragged
@pytest.mark.parametrize("N,T,K_in,K_out,kept,jacobian", [
    (9, 215, 456, 40, 9, False), (9, 215, 456, 64, 9, True), (9, 215, 456, 72, 9, False), (9, 215, 456, 200, 9, True),
    (12, 215, 456, 72, 9, True), (5, 413, 1000, 8, 5, False), (5, 413, 1000, 136, 4, True), (5, 413, 1000, 256, 5, False),
    (5, 413, 1000, 264, 5, True), (5, 413, 1000, 320, 5, False), (5, 413, 1000, 328, 5, False), (5, 413, 1000, 776, 5, False),
    (5, 413, 2056, 128, 5, True), (5, 413, 2056, 192, 5, False), (5, 413, 2056, 264, 4, False), (5, 413, 2056, 328, 5, False), (4, 512, 1024, 136, 4, False), (40, 13, 4040, 24, 37, True), (33, 64, 1040, 72, 1, False)])
def test_fp32_dgrad_tiles(vb, N, T, K_in, K_out, kept, jacobian):
    R = N * T
    shape = vb.shape_of(N, T, K_in, K_out, vb.VCAS_F32)
    gen = torch.Generator(device="cuda").manual_seed(K_out + kept)
    G = torch.randn((R, K_out), generator=gen, device="cuda")
    W = torch.randn((K_out, K_in), generator=gen, device="cuda") * 0.02
    J = torch.rand((R, K_in), generator=gen, device="cuda")
    p = torch.rand(N, generator=gen, device="cuda") * 0.5 + 0.5
    chosen = torch.randperm(N, generator=gen, device="cuda")[:kept].sort().values
    idxA = torch.full((N,), -1, dtype=torch.int32, device="cuda")
    idxA[:kept] = chosen.int()
    cntA = torch.tensor([kept], dtype=torch.int32, device="cuda")
    rows = torch.zeros(N, device="cuda")
    rows[chosen] = 1.0 / p[chosen]
    rows = rows.repeat_interleave(T)[:, None]
    G[rows[:, 0] == 0] = float("nan")    # rows of dropped samples are not read
    dX = torch.full((R, K_in), float("nan"), device="cuda")
    if jacobian:
        vb.vcas_sampled_dgrad_jac(shape, G, W, p, idxA, cntA, J, dX)
    else:
        vb.vcas_sampled_dgrad(shape, G, W, p, idxA, cntA, dX)
    want = (G.nan_to_num().double() @ W.double()) * rows.double() * (J.double() if jacobian else 1.0)
    on = rows[:, 0] > 0
    assert float(dX[~on].abs().sum()) == 0.0
    off = (dX.double() - want)[on]
    # sums of up to 776 fp32 products: sqrt(776) 2^-24 = 2e-6, a row or a column alike
    assert float((off.norm(dim=1) / want[on].norm(dim=1)).max()) <= 1e-5
    assert float((off.norm(dim=0) / want[on].norm(dim=0)).max()) <= 1e-5


# bf16 dgrad on both sides of the contraction length from which it reads whole steps ahead (512: eight steps), full and
# ragged last steps, 64x128 and 128x128 tiles of either kind; 243 and 261 tiles of 64x128, about one to a CU
@pytest.mark.parametrize("K_out", [8, 64, 72, 128, 136, 504, 512, 520, 568, 576, 640, 1032])
@pytest.mark.parametrize("N,T,K_in", [(5, 41, 200), (9, 233, 776), (11, 233, 1544), (13, 130, 1128), (13, 140, 1128)])
def test_bf16_dgrad_contractions(vb, N, T, K_in, K_out):
    R = N * T
    shape = vb.shape_of(N, T, K_in, K_out, vb.VCAS_BF16)
    gen = torch.Generator(device="cuda").manual_seed(K_out + N)
    G = torch.randn((R, K_out), generator=gen, device="cuda").bfloat16()
    W = (torch.randn((K_out, K_in), generator=gen, device="cuda") * 0.02).bfloat16()
    J = torch.rand((R, K_in), generator=gen, device="cuda").bfloat16()
    p = torch.rand(N, generator=gen, device="cuda") * 0.5 + 0.5
    idxA = torch.arange(1, N + 1, dtype=torch.int32, device="cuda")      # all samples but the first
    cntA = torch.tensor([N - 1], dtype=torch.int32, device="cuda")
    G[:T] = float("nan")    # rows of dropped samples are not read
    dX = torch.full((R, K_in), float("nan"), dtype=torch.bfloat16, device="cuda")
    vb.vcas_sampled_dgrad_jac(shape, G, W, p, idxA, cntA, J, dX)
    want = (G[T:].double() @ W.double()) / p[1:].double().repeat_interleave(T)[:, None] * J[T:].double()
    assert float(dX[:T].abs().sum()) == 0.0
    off = dX[T:].double() - want
    # fp32 sums rounded once to bf16: 2^-9 / sqrt(3) = 1.1e-3; a row or a column alike
    assert float((off.norm(dim=1) / want.norm(dim=1)).max()) <= 5e-3
    assert float((off.norm(dim=0) / want.norm(dim=0)).max()) <= 5e-3


# The quartered last round as an entry of a stack reaches it: dropped rows left unwritten (a grid without zero-fill duty) or
# zeroed, SampleA ahead of dgrad, inside it from the row sums (up to 4096 rows) and from the lane sums of block sums, where a
# workgroup's second quarter goes on with the kept list in LDS; a list of more than the 1024 samples that are staged.
# Whole 256x256 tiles in front of the quarters, one quarter to a workgroup (up to 64 tiles), two (up to 128).
@pytest.mark.parametrize("N,T,K_in,K_out,rho,live,draw,whole,tail,route", [
    (40, 257, 1608, 1544, 1.0, 40, 0, 256, 31, "swept"), (40, 257, 1608, 1544, 1.0, 40, 0, 256, 31, "blocks"),
    (40, 257, 1352, 1544, 0.5, 40, 0, 0, 126, "swept"), (40, 257, 1352, 1544, 0.5, 40, 0, 0, 126, "blocks"),
    (40, 257, 1352, 1536, 0.5, 9, 0, 0, 60, "swept"), (40, 257, 1352, 1536, 0.5, 9, 0, 0, 60, "blocks"),
    (64, 64, 4040, 1544, 0.6, 64, 9, 0, 128, "swept"), (64, 64, 4040, 1544, 0.6, 15, 0, 0, 64, "swept"),
    (64, 64, 4040, 1544, 0.6, 64, 9, 0, 128, "blocks"), (1100, 9, 1608, 1544, 1.0, 1100, 0, 256, 17, "swept")])
@pytest.mark.parametrize("fill", [False, True])
def test_quarters_of_a_stack_entry(vb, N, T, K_in, K_out, rho, live, draw, whole, tail, route, fill):
    R = N * T
    shape = vb.shape_of(N, T, K_in, K_out, vb.VCAS_BF16)
    gen = torch.Generator(device="cuda").manual_seed(N + live)
    G = torch.randn((R, K_out), generator=gen, device="cuda").bfloat16()
    G.mul_(torch.linspace(1.0, 1.5, N, device="cuda").bfloat16().repeat_interleave(T)[:, None])
    X = torch.randn((R, K_in), generator=gen, device="cuda").bfloat16()
    W = (torch.randn((K_out, K_in), generator=gen, device="cuda") * 0.02).bfloat16()
    above = torch.zeros(N, dtype=torch.uint8, device="cuda")
    above[torch.randperm(N, generator=gen, device="cuda")[:live]] = 1
    gone = above.repeat_interleave(T) == 0
    G[gone] = float("nan")    # never read
    groups = (K_out + 255) // 256
    squares = torch.zeros((R, groups * 256), device="cuda")
    squares[:, :K_out] = G.nan_to_num().float().square()
    blocks = squares.view(R, groups, 4, 64).sum(3).permute(1, 0, 2).contiguous()
    plan, ws = vb.Plan.allocate(N, T), vb.make_workspace(shape)
    dX = torch.full((R, K_in), float("nan"), dtype=torch.bfloat16, device="cuda")
    entry = vb.layer_args(shape, G, X, W, rho, 0.5, vb.Rng(7, 1, draw), True, plan, dX, None, ws, kept_above=above,
                          leave_dropped_rows=not fill, g_sq_blocks=blocks if route == "blocks" else None)
    vb.vcas_backward_stack(vb.make_stack([entry]), 1, torch.cuda.Stream(), torch.cuda.Stream())
    torch.cuda.synchronize()
    norms = torch.where(gone, 0.0, G.nan_to_num().double().square().sum(1)).view(N, T).sum(1).sqrt()
    assert float((plan.gnorm.double() - norms).abs().max() / norms.max()) <= 1e-5
    mask, p = plan.maskA.bool(), plan.p
    kept = int(mask.sum())
    tiles = (kept * T + 255) // 256 * ((K_in + 255) // 256)
    assert tiles == whole + tail, (kept, tiles)     # the case is what it says
    assert bool((mask <= above.bool()).all()) and kept == int(plan.cntA.item())
    on = mask.repeat_interleave(T)
    want = (G[on].double() @ W.double()) / p[mask].double().repeat_interleave(T)[:, None]
    off = dX[on].double() - want
    # fp32 sums rounded once to bf16: 2^-9 / sqrt(3) = 1.1e-3; a row or a column alike
    assert float((off.norm(dim=1) / want.norm(dim=1)).max()) <= 5e-3
    assert float((off.norm(dim=0) / want.norm(dim=0)).max()) <= 5e-3
    rest = dX[~on]
    assert bool((rest == 0).all()) if fill else bool(torch.isnan(rest).all())


def test_dgrad_tile_where_few_tiles_cannot_become_a_second_round(vb):
    """207 tiles of 64x128 are expected, 243 are all there can be: one to a CU, half the rows of the 128x128 tile.  The larger
    tile (99 of them at work) took 1.2 times as long."""
    N, T, K_in, K_out = 13, 130, 1128, 3376
    R = N * T
    shape = vb.shape_of(N, T, K_in, K_out, vb.VCAS_BF16)
    G = torch.randn((R, K_out), device="cuda").bfloat16()
    X = torch.randn((R, K_in), device="cuda").bfloat16()
    W = torch.randn((K_out, K_in), device="cuda").bfloat16()
    plan, ws = vb.Plan.allocate(N, T), vb.make_workspace(shape)
    dX = torch.empty((R, K_in), dtype=torch.bfloat16, device="cuda")

    def per_launch(rho):
        vb.vcas_backward_data(shape, G, X, W, rho, vb.Rng(1, 1, 0), True, plan, dX, ws)
        torch.cuda.synchronize()
        vb.vcas_profile_begin()
        for draw in range(40):
            vb.vcas_backward_data(shape, G, X, W, rho, vb.Rng(1, 1, draw), True, plan, dX, ws)
        return vb.vcas_profile_end()[0][0] / 40

    expected_200_at_most = min(per_launch(0.8) for _ in range(3))    # 198 tiles
    assert min(per_launch(0.834) for _ in range(3)) <= 1.1 * expected_200_at_most


def test_fp32_dgrad_of_a_ragged_contraction(vb):
    """8 x 26 tiles of 128x128: a contraction of 272 takes less than one of 320 (nine steps of 32 and ten; in steps of 64 it took 0.99
    of it)."""
    N, T, K_in = 8, 121, 3264
    R = N * T

    def took(K):
        shape = vb.shape_of(N, T, K_in, K, vb.VCAS_F32)
        G, W, dX = torch.randn((R, K), device="cuda"), torch.randn((K, K_in), device="cuda"), torch.empty((R, K_in), device="cuda")
        p, cnt = torch.ones(N, device="cuda"), torch.tensor([N], dtype=torch.int32, device="cuda")
        idx = torch.arange(N, dtype=torch.int32, device="cuda")
        best = float("inf")
        for _ in range(4):
            vb.vcas_profile_begin()
            for _ in range(20):
                vb.vcas_sampled_dgrad(shape, G, W, p, idx, cnt, dX)
            best = min(best, vb.vcas_profile_end()[0][0] / 20)
        return best

    assert took(272) <= 0.97 * took(320)
