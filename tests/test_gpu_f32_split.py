"""fp32 products from bf16 parts: the lines between the tiles of the weight gradient and the edges of its slices, the accuracy
that three parts and separate small sums give, operands down to fp32's smallest numbers, and operands whose parts are not finite, against
64 bits."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vb():
    from paper_2402_17227_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


def _wgrad(vb, G, X, scale, kept):
    R = G.shape[0]
    shape = vb.shape_of(1, R, X.shape[1], G.shape[1], vb.VCAS_F32)
    idx = torch.full((R,), -1, dtype=torch.int32, device="cuda")
    idx[:len(kept)] = kept.int()
    cnt = torch.tensor([len(kept)], dtype=torch.int32, device="cuda")
    dW = torch.full((G.shape[1], X.shape[1]), float("nan"), device="cuda")
    vb.vcas_sampled_wgrad(shape, G, X, scale, idx, cnt, dW, vb.make_workspace(shape))
    return dW


def _bound(k):
    # left out of a product: 2^-24 of it at the most; sums rounded once per 16 terms: sqrt(k / 16) 2^-24 (one wavefront's part of
    # the contraction and the slices have fewer)
    return (math.sqrt(k / 16) + 2) * 2.0 ** -24


# 64x64 tiles (from 65 of them, 101 for few tokens), then, from about 1250 rows on, 128x128 tiles in eight slices: all active, some, one, none;
# steps of 64 and of 32 tokens that are full, ragged, single; 128x128 tiles from 257 of 64x64 up, whole up to some 600 tokens, in two
# and three slices beyond, whole at any number from 129 of them up
@pytest.mark.parametrize("R,K_in,K_out,kept", [
    (1200, 520, 520, 1200), (1200, 520, 584, 65), (700, 584, 520, 1), (700, 520, 520, 0), (192, 520, 520, 64), (140, 776, 520, 140),
    (4001, 520, 520, 4001), (4001, 520, 584, 1025), (4001, 584, 520, 1023), (4001, 520, 520, 257), (4001, 520, 520, 129),
    (4001, 520, 520, 127), (4001, 520, 520, 1), (4001, 520, 520, 0), (1500, 768, 768, 1500),
    (300, 1288, 1160, 300), (300, 1160, 1288, 33), (300, 1288, 1160, 31), (40, 1288, 1160, 1),
    (300, 776, 1544, 300), (1500, 1288, 1160, 1500), (1500, 1160, 1288, 257), (1500, 1288, 1160, 127), (1200, 776, 1416, 1111), (1500, 1288, 1672, 1500)])
def test_wgrad_tiles_and_slices(vb, R, K_in, K_out, kept):
    gen = torch.Generator(device="cuda").manual_seed(R + kept)
    G = torch.randn((R, K_out), generator=gen, device="cuda")
    X = torch.randn((R, K_in), generator=gen, device="cuda")
    scale = torch.rand(R, generator=gen, device="cuda") * 3 + 1
    rows = torch.randperm(R, generator=gen, device="cuda")[:kept].sort().values
    on = torch.zeros(R, dtype=torch.bool, device="cuda")
    on[rows] = True
    G[~on], X[~on] = float("nan"), float("inf")    # tokens that are not kept are not read
    dW = _wgrad(vb, G, X, scale, rows).double()
    want = (G[rows] * scale[rows, None]).double().t() @ X[rows].double()   # the scaled operand is rounded once, as in the library
    if not kept:
        assert float(dW.abs().sum()) == 0.0
        return
    for dim in (0, 1):
        assert float(((dW - want).norm(dim=dim) / want.norm(dim=dim)).max()) <= 4 * _bound(kept)   # a row has its own spread
    assert float((dW - want).norm() / want.norm()) <= _bound(kept)


# One kept token: a product rounded once, as on the fp32 instruction, and not the 9e-8 that the parts leave; few tokens no
# more than fp32 sums of that many terms
@pytest.mark.parametrize("kept", [1, 2, 3, 7])
@pytest.mark.parametrize("R,K_in,K_out", [(700, 584, 776), (4001, 520, 520), (300, 1288, 1160), (40, 1288, 2056)])
def test_wgrad_of_few_tokens(vb, R, K_in, K_out, kept):
    gen = torch.Generator(device="cuda").manual_seed(R)
    G = torch.randn((R, K_out), generator=gen, device="cuda")
    X = torch.randn((R, K_in), generator=gen, device="cuda")
    scale = torch.ones(R, device="cuda")
    rows = torch.arange(kept, device="cuda") * 5 + 2
    dW = _wgrad(vb, G, X, scale, rows).double()
    g, x = G[rows].double(), X[rows].double()
    off = (dW - g.t() @ x).abs()
    terms = g.abs().t() @ x.abs()
    # a rounding of the sum so far with every term
    assert float((off / terms).max()) <= kept * 2.0 ** -24


# every tile of the data half: 64x64, 64x128, 128x128
@pytest.mark.parametrize("R,K_in,K_out", [(1935, 456, 200), (1100, 1000, 776), (2065, 2056, 328)])
def test_dgrad_accuracy(vb, R, K_in, K_out):
    gen = torch.Generator(device="cuda").manual_seed(R)
    G = torch.randn((R, K_out), generator=gen, device="cuda")
    W = torch.randn((K_out, K_in), generator=gen, device="cuda") * 0.02
    dX = _dgrad(vb, G, W).double()
    want = G.double() @ W.double()
    assert float((dX - want).norm() / want.norm()) <= _bound(K_out)


def _dgrad(vb, G, W):
    R = G.shape[0]
    ones = torch.ones(1, device="cuda")
    zero, one = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.ones(1, dtype=torch.int32, device="cuda")
    dX = torch.full((R, W.shape[1]), float("nan"), device="cuda")
    vb.vcas_sampled_dgrad(vb.shape_of(1, R, W.shape[1], W.shape[0], vb.VCAS_F32), G, W, ones, zero, one, dX)
    return dX


# Operands of about 2^a and 2^b: values whose small parts are below bf16's smallest number, subnormal ones, products whose small
# parts are; values and sums that are beyond what the parts can hold
RANGES = [(-112, 30), (-118, 30), (-126, 60), (-140, 60), (30, -126), (-60, -60), (106, -100), (45, 45)]


@pytest.mark.parametrize("a,b", RANGES)
@pytest.mark.parametrize("R,K_in,K_out", [(1935, 456, 200), (1100, 1000, 776), (2065, 2056, 328)])
def test_dgrad_keeps_small_values(vb, R, K_in, K_out, a, b):
    gen = torch.Generator(device="cuda").manual_seed(R)
    G = (torch.randn((R, K_out), generator=gen, device="cuda").double() * 2.0 ** a).float()
    W = (torch.randn((K_out, K_in), generator=gen, device="cuda").double() * 2.0 ** b).float()
    off, want = _dgrad(vb, G, W).double(), G.double() @ W.double()
    off -= want
    for dim in (0, 1):
        assert float((off.norm(dim=dim) / want.norm(dim=dim)).max()) <= 4 * _bound(K_out)


@pytest.mark.parametrize("a,b", RANGES)
@pytest.mark.parametrize("R,K_in,K_out", [(1200, 520, 520), (4001, 520, 520), (300, 1288, 1160)])
def test_wgrad_keeps_small_values(vb, R, K_in, K_out, a, b):
    gen = torch.Generator(device="cuda").manual_seed(R)
    G = (torch.randn((R, K_out), generator=gen, device="cuda").double() * 2.0 ** a).float()
    X = (torch.randn((R, K_in), generator=gen, device="cuda").double() * 2.0 ** b).float()
    scale = torch.full((R,), 4.0, device="cuda")
    off, want = _wgrad(vb, G, X, scale, torch.arange(R, device="cuda")).double(), 4 * (G.double().t() @ X.double())
    off -= want
    for dim in (0, 1):
        assert float((off.norm(dim=dim) / want.norm(dim=dim)).max()) <= 4 * _bound(R)


def _same(got, A, B):
    """got = A B: infinities, NaN and numbers in the same places, and numbers within fp32 sums of their terms."""
    A, B = A.double(), B.double()
    want = A @ B
    terms = A.nan_to_num(0, 0, 0).abs() @ B.nan_to_num(0, 0, 0).abs()
    assert torch.equal(got.isnan(), want.isnan())
    assert torch.equal(got.isposinf(), want.isposinf()) and torch.equal(got.isneginf(), want.isneginf())
    ok = want.isfinite()
    assert float(((got - want).abs() / terms)[ok].max()) <= 1e-6


def _spoil(A, B):
    """Values that bf16 parts cannot hold into a few rows of A [k, m] and B [k, n]: infinities that meet numbers whose small
    parts are zero, a NaN, and the largest finite value, which rounds to infinity in bf16."""
    A[3, 5], A[70, 17] = float("inf"), float("-inf")
    B[3], B[70] = 0.5, -2.0          # exact in bf16: their other parts are zero
    A[11, 40] = float("nan")
    A[12, 41] = 3.4e38
    B[12] = B[12] * 1e-3
    B[20, 9] = float("inf")
    A[20] = A[20].abs() + 0.25
    B[21, 33] = -3.4e38
    A[21] = A[21] * 1e-3


@pytest.mark.parametrize("R,K_in,K_out", [(1935, 456, 200), (1100, 1000, 776), (2065, 2056, 328)])
def test_dgrad_of_values_without_finite_parts(vb, R, K_in, K_out):
    gen = torch.Generator(device="cuda").manual_seed(K_out)
    G = torch.randn((R, K_out), generator=gen, device="cuda")
    W = torch.randn((K_out, K_in), generator=gen, device="cuda")
    Gt = G.t().contiguous()
    _spoil(Gt, W)
    G = Gt.t().contiguous()
    _same(_dgrad(vb, G, W).double(), G, W)


@pytest.mark.parametrize("R,K_in,K_out", [(1200, 520, 520), (4001, 520, 520), (300, 1288, 1160)])
def test_wgrad_of_values_without_finite_parts(vb, R, K_in, K_out):
    gen = torch.Generator(device="cuda").manual_seed(K_out)
    G = torch.randn((R, K_out), generator=gen, device="cuda")
    X = torch.randn((R, K_in), generator=gen, device="cuda")
    _spoil(G, X)
    scale = torch.ones(R, device="cuda")
    _same(_wgrad(vb, G, X, scale, torch.arange(R, device="cuda")).double(), G.t(), X)
