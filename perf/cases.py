"""Performance cases of the sampled linear-layer backward: what a training program has this library do.

Four kinds of work, all through the public binding:

  layer   one vcas_linear_backward call: row norms, SampleA, dX, SampleW, dW of one linear layer, on one
          stream or with the weight half on a side stream that the caller joins;
  halves  the same layer as a framework's autograd would call it, the two halves apart: the data half with the
          Jacobian of the elementwise layer below and the samples dropped above
          (vcas_backward_data_chained), then the weight half on the cached norms of X
          (vcas_backward_weight_cached);
  stack   a stack of encoder blocks (down, up, o, then V, K and Q together) in one vcas_backward_stack call over
          three streams, every dX the next entry's G;
  adapt   what one layer costs in an update of the adaptive keep ratios: the exact backward, its running
          statistics, the variance probe over M mask draws and the sparsity at two levels.

Values: X ~ N(0,1), W ~ N(0, 0.02^2), G = per-sample LogNormal scale * per-token LogNormal scale * N(0,1), as in
workloads.py.  A listed case's sizes are those of workloads.py where its comment names one.
"""
from __future__ import annotations

import math

import torch

from paper_2402_17227_amd import binding as vb

BF16, F32 = "bf16", "f32"


def _layer(name, dtype, N, T, K_in, K_out, rho, nu, sample_sigma, token_sigma, side):
    return dict(name=name, kind="layer", dtype=dtype, N=N, T=T, K_in=K_in, K_out=K_out, rho=rho, nu=nu,
                sample_sigma=sample_sigma, token_sigma=token_sigma, side=side)


def _stack(name, N, T, hidden, ffn, blocks, rho_top, rho_bottom, nu, sample_sigma, token_sigma, jacobian, cached):
    return dict(name=name, kind="stack", dtype=BF16, N=N, T=T, hidden=hidden, ffn=ffn, blocks=blocks, rho_top=rho_top,
                rho_bottom=rho_bottom, nu=nu, sample_sigma=sample_sigma, token_sigma=token_sigma, jacobian=jacobian,
                cached=cached)


def listed():
    return [
        # A small head or adapter with ragged sizes (the tests' ragged case): launches and latency.
        _layer("tiny ragged bf16", BF16, 5, 37, 264, 136, 0.6, 0.5, 1.0, 0.5, False),
        # The single fp32 layer of workloads.py.
        _layer("single f32", F32, 8, 128, 768, 768, 0.5, 0.5, 1.0, 0.0, False),
        # A feed-forward layer at finetuning size in full precision.
        _layer("base ffn f32", F32, 32, 128, 768, 3072, 0.5, 0.5, 1.0, 0.5, False),
        # The feed-forward layer of bert_base, called on its own on one stream.
        _layer("base ffn bf16", BF16, 32, 128, 768, 3072, 0.5, 0.5, 1.0, 0.5, False),
        # An attention projection of bert_large, the weight half on a side stream.
        _layer("large proj bf16 side", BF16, 32, 512, 1024, 1024, 0.25, 0.4, 1.0, 0.5, True),
        # A large pretraining batch, 64 Ki tokens on one GPU.
        _layer("64k-token ffn bf16", BF16, 64, 1024, 1024, 4096, 0.5, 0.5, 0.0, 0.5, False),
        # vit_b16's second feed-forward layer (197 tokens: nothing divides), the halves apart.
        dict(name="vit ffn halves bf16", kind="halves", dtype=BF16, N=64, T=197, K_in=3072, K_out=768, rho=0.3, nu=0.5,
             sample_sigma=1.5, token_sigma=0.0),
        # The whole bert_base stack.
        _stack("base stack bf16", 32, 128, 768, 3072, 12, 1.0, 0.3, 0.5, 1.0, 0.5, False, False),
        # Four blocks of bert_large over the whole range of its keep ratios.
        _stack("large stack bf16", 32, 512, 1024, 4096, 4, 1.0, 0.25, 0.4, 1.0, 0.5, False, False),
        # Two blocks of gpt2_medium through their activation's Jacobian, the norms of X kept from the forward pass.
        _stack("gpt2 stack bf16", 16, 1024, 1024, 4096, 2, 0.5, 0.5, 0.5, 0.0, 0.5, True, True),
        # The probe of vit_b16: eight mask draws.
        dict(name="vit adapt bf16", kind="adapt", dtype=BF16, N=64, T=197, K_in=768, K_out=768, rho=0.3, nu=0.5,
             sample_sigma=1.5, token_sigma=0.0, M=8),
        # An update in full precision with the paper's M = 2.
        dict(name="small adapt f32", kind="adapt", dtype=F32, N=16, T=128, K_in=768, K_out=768, rho=0.5, nu=0.5,
             sample_sigma=1.0, token_sigma=0.5, M=2),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _width(rng, lo, hi):
    """A row length: a multiple of 8, as the library wants, a multiple of 64 half of the time."""
    step = rng.choice((8, 64))
    return max(step, _log_int(rng, lo, hi) // step * step)


def draw(rng):
    """One more case of the same ranges: 1 to 128 samples of 1 to 1024 tokens, rows of 64 to 4096 elements, keep
    ratios of 0.2 to 1, every kind, type and option above."""
    kind = rng.choice(("layer", "layer", "layer", "layer", "halves", "stack", "stack", "adapt"))
    case = dict(kind=kind, dtype=F32 if kind != "stack" and rng.random() < 0.35 else BF16)
    # multiply-adds of one dense product that the case may have: those of the largest listed case of its kind
    most = {"stack": 16384 * 1024 * 4096, "adapt": 64 * 197 * 768 * 768}.get(kind, 65536 * 1024 * 4096)
    if case["dtype"] == F32:
        most = {"adapt": 16 * 128 * 768 * 768}.get(kind, 32 * 128 * 768 * 3072)
    if kind == "stack":
        case.update(hidden=64 * rng.randint(4, 16), blocks=rng.randint(1, 4))
        case["ffn"] = case["hidden"] * rng.choice((2, 3, 4))
        widest = case["hidden"] * case["ffn"]
    else:
        case.update(K_in=_width(rng, 64, 4096), K_out=_width(rng, 64, 4096))
        widest = case["K_in"] * case["K_out"]
    while True:
        N, T = _log_int(rng, 1, 128), _log_int(rng, 1, 1024)
        if N * T * widest <= most and N * T <= (16384 if kind == "stack" else 65536) and N * T >= 64:
            break
        if 64 * widest > most:
            case["K_in"] = widest = 64
            widest *= case["K_out"]
    case.update(N=N, T=T, nu=round(rng.uniform(0.2, 1.0), 3), sample_sigma=rng.choice((0.0, 1.0, 1.5)),
                token_sigma=rng.choice((0.0, 0.5)))
    if kind == "stack":
        case.update(rho_top=round(rng.uniform(0.5, 1.0), 3), rho_bottom=round(rng.uniform(0.2, 0.5), 3),
                    jacobian=rng.random() < 0.5, cached=rng.random() < 0.5)
    else:
        case["rho"] = round(rng.uniform(0.2, 1.0), 3)
    if kind == "layer":
        case["side"] = rng.random() < 0.5
    if kind == "adapt":
        case["M"] = rng.randint(2, 8 if case["dtype"] == BF16 else 2)
    return case


class _Inputs:
    """Seeded tensors on the GPU, in the layer's type."""

    def __init__(self, case, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(seed)
        self.dtype = torch.bfloat16 if case["dtype"] == BF16 else torch.float32
        self.code = vb.VCAS_BF16 if case["dtype"] == BF16 else vb.VCAS_F32
        self.N, self.T, self.seed = case["N"], case["T"], seed
        self.sigmas = case["sample_sigma"], case["token_sigma"]

    def normal(self, *size, dtype=None):
        return torch.randn(size, generator=self.gen, device="cuda", dtype=dtype or self.dtype)

    def weight(self, K_out, K_in):
        return self.normal(K_out, K_in).mul_(0.02)

    def gradient(self, K_out):
        s = torch.exp(self.sigmas[0] * self.normal(self.N, 1, dtype=torch.float32))
        t = torch.exp(self.sigmas[1] * self.normal(self.N, self.T, dtype=torch.float32))
        return self.normal(self.N * self.T, K_out).mul_((s * t).to(self.dtype).view(-1, 1))

    def jacobian(self, K_in):
        """Derivative of a GELU at normal inputs."""
        z = self.normal(self.N * self.T, K_in)
        return torch.sigmoid(z.mul_(1.702)).add_(z.mul_(0.1).clamp_(-0.2, 0.2))

    def row_norms(self, shape, X):
        out = torch.empty(self.N * self.T, device="cuda")
        vb.vcas_row_norms(shape, None, X, None, None, out, None)
        return out


def _plan_outputs(plan):
    # idxA and idxW hold their counts' worth of entries only, which the masks give too
    return [plan.gsq, plan.gnorm, plan.p, plan.maskA, plan.cntA, plan.xsq, plan.score, plan.q, plan.maskW, plan.cntW,
            plan.scaleW]


def _prepare_single(case, inp):
    K_in, K_out, R = case["K_in"], case["K_out"], case["N"] * case["T"]
    st = dict(kind=case["kind"], rho=case["rho"], nu=case["nu"], rng=vb.Rng(inp.seed, 3, 0))
    st["shape"] = vb.shape_of(case["N"], case["T"], K_in, K_out, inp.code)
    st.update(G=inp.gradient(K_out), X=inp.normal(R, K_in), W=inp.weight(K_out, K_in), plan=vb.Plan.allocate(case["N"], case["T"]),
              ws=vb.make_workspace(st["shape"]), dX=torch.empty((R, K_in), dtype=inp.dtype, device="cuda"),
              dW=torch.empty((K_out, K_in), device="cuda"))
    if case["kind"] == "layer":
        st["side"] = torch.cuda.Stream() if case["side"] else None
    elif case["kind"] == "halves":
        # one sample in four was dropped by the layers above
        above = (torch.arange(case["N"], device="cuda") % 4 != 3).to(torch.uint8)
        st.update(J=inp.jacobian(K_in), kept_above=above, xsq=inp.row_norms(st["shape"], st["X"]))
    else:
        n, stride = K_out * K_in, 100        # App. D: every 100th parameter
        m = (n + stride - 1) // stride
        st.update(M=case["M"], m=m, stride=stride, mean=torch.zeros(m, device="cuda"), sqmean=torch.zeros(m, device="cuda"),
                  probe=torch.zeros(4, dtype=torch.float64, device="cuda"), sparsity=torch.zeros(2, device="cuda"))
    return st


def _rho(case, b):
    f = b / (case["blocks"] - 1) if case["blocks"] > 1 else 1.0
    return case["rho_bottom"] + (case["rho_top"] - case["rho_bottom"]) * f


def _entries(case):
    """(name, K_in, K_out, rho) in backward order: the top block first."""
    h, f = case["hidden"], case["ffn"]
    for b in reversed(range(case["blocks"])):
        for name, K_in, K_out in (("down", f, h), ("up", h, f), ("o", h, h), ("v", h, h), ("k", h, h), ("q", h, h)):
            yield name, K_in, K_out, _rho(case, b)


def _prepare_stack(case, inp):
    """As a training program keeps it: one buffer for the gradients of all weights, one for those of all
    activations, one per field of the plans."""
    N, T, R = case["N"], case["T"], case["N"] * case["T"]
    layers = list(_entries(case))
    L = len(layers)
    f32 = dict(dtype=torch.float32, device="cuda")
    u8 = dict(dtype=torch.uint8, device="cuda")
    i32 = dict(dtype=torch.int32, device="cuda")
    field = dict(gsq=torch.zeros((L, R), **f32), gnorm=torch.zeros((L, N), **f32), p=torch.zeros((L, N), **f32),
                 maskA=torch.zeros((L, N), **u8), idxA=torch.zeros((L, N), **i32), cntA=torch.zeros((L, 1), **i32),
                 xsq=torch.zeros((L, R), **f32), score=torch.zeros((L, R), **f32), q=torch.zeros((L, R), **f32),
                 maskW=torch.zeros((L, R), **u8), idxW=torch.zeros((L, R), **i32), cntW=torch.zeros((L, 1), **i32),
                 scaleW=torch.zeros((L, R), **f32))
    dW = torch.zeros(sum(K_in * K_out for _, K_in, K_out, _ in layers), **f32)
    # zeroed once: the rows of samples that a layer drops are never written
    dX = torch.zeros(sum(R * K_in for _, K_in, _, _ in layers), dtype=inp.dtype, device="cuda")
    st = dict(kind="stack", field=field, dW=dW, dX=dX, keep=[], group=3 if R <= 4096 else 6,
              streams=(torch.cuda.Stream(), torch.cuda.Stream()))
    entries, at_w, at_x = [], 0, 0
    G, above = inp.gradient(layers[0][2]), None
    st["keep"].append(G)
    for l, (name, K_in, K_out, rho) in enumerate(layers):
        shape = vb.shape_of(N, T, K_in, K_out, inp.code)
        plan = vb.Plan(**{k: v[l] for k, v in field.items()})
        X, W, ws = inp.normal(R, K_in), inp.weight(K_out, K_in), vb.make_workspace(shape)
        J = inp.jacobian(K_in) if case["jacobian"] and name == "down" else None
        xsq = inp.row_norms(shape, X) if case["cached"] else None
        my_dW, my_dX = dW[at_w:at_w + K_in * K_out], dX[at_x:at_x + R * K_in]
        at_w, at_x = at_w + K_in * K_out, at_x + R * K_in
        sibling = name in ("k", "q")         # K and Q take the G that V took
        entries.append(vb.layer_args(shape, G, X, W, rho, case["nu"], vb.Rng(inp.seed, l, 0), True, plan, my_dX, my_dW, ws,
                                     xsq_forward=xsq, sibling=sibling, J=J, kept_above=above, leave_dropped_rows=True,
                                     wgrad_fill=64))
        st["keep"].append((X, W, ws, J, xsq, plan))
        if name in ("down", "up", "q"):
            G, above = my_dX, plan.maskA
        elif name == "o":
            G, above = my_dX, plan.maskA
    st["stack"] = vb.make_stack(entries)
    return st


def prepare(case, seed):
    inp = _Inputs(case, seed)
    return _prepare_stack(case, inp) if case["kind"] == "stack" else _prepare_single(case, inp)


def run(st):
    kind = st["kind"]
    main = torch.cuda.current_stream()
    if kind == "stack":
        s2, s3 = st["streams"]
        vb.vcas_backward_stack(st["stack"], st["group"], s2, s3)
        main.wait_stream(s2)
        main.wait_stream(s3)
        f = st["field"]
        # scaleW follows from p, q and maskW
        return [st["dX"], st["dW"]] + [f[k] for k in ("gsq", "gnorm", "p", "maskA", "cntA", "xsq", "score", "q", "maskW",
                                                       "cntW")]
    shape, G, X, W, plan, ws, rho, nu, rng = (st[k] for k in ("shape", "G", "X", "W", "plan", "ws", "rho", "nu", "rng"))
    dX, dW = st["dX"], st["dW"]
    if kind == "layer":
        side = st["side"]
        vb.vcas_linear_backward(shape, G, X, W, rho, nu, rng, True, plan, dX, dW, ws, side)
        if side is not None:
            main.wait_stream(side)
        return [dX, dW] + _plan_outputs(plan)
    if kind == "halves":
        vb.vcas_backward_data_chained(shape, G, X, W, st["J"], st["kept_above"], True, rho, rng, True, plan, dX, ws)
        vb.vcas_backward_weight_cached(shape, G, X, st["xsq"], rho, nu, rng, True, plan, dW, ws)
        return [dX, dW] + _plan_outputs(plan)
    vb.vcas_linear_backward(shape, G, X, W, 1.0, 1.0, rng, True, plan, dX, dW, ws)
    vb.vcas_grad_stats_update(dW, st["m"], st["stride"], 1, st["mean"], st["sqmean"])
    vb.vcas_variance_probe(shape, G, X, rho, nu, rng, st["M"], plan, st["probe"], ws)
    vb.vcas_sparsity_ratio(plan.gnorm, [0.98, 1.0], st["sparsity"])
    return [dX, dW, st["mean"], st["sqmean"], st["probe"], st["sparsity"]] + _plan_outputs(plan)


def _layer_work(R, K_in, K_out, e, rho, nu, dx_rows, g_rows, x_rows):
    """G for its norms, X of kept samples, W, dX, dW and the plan's vectors once each; products over kept rows."""
    nbytes = e * (g_rows * K_out + x_rows * K_in + K_in * K_out + dx_rows * K_in) + 4 * K_in * K_out + 29 * R
    return nbytes, 2.0 * R * K_in * K_out * (rho + rho * nu)


def work(case):
    R, e = case["N"] * case["T"], 2 if case["dtype"] == BF16 else 4
    nbytes = flops = 0.0
    if case["kind"] == "stack":
        above = 1.0      # the rows of G that exist: those of the samples the layer above kept
        for name, K_in, K_out, rho in _entries(case):
            # cached norms of X: only kept tokens' rows of X are read, for dW
            x_share = rho * case["nu"] if case["cached"] else rho
            b, f = _layer_work(R, K_in, K_out, e, rho, case["nu"], rho * R, (0 if name in ("k", "q") else above) * R, x_share * R)
            nbytes += b + (rho * R * K_in * e if case["jacobian"] and name == "down" else 0) + (4 * R if case["cached"] else 0)
            flops += f
            above = min(above, rho) if name not in ("v", "k") else above
        return {"bytes": nbytes, "flops": flops}
    rho, nu, K_in, K_out = case["rho"], case["nu"], case["K_in"], case["K_out"]
    if case["kind"] == "layer":
        nbytes, flops = _layer_work(R, K_in, K_out, e, rho, nu, R, R, rho * R)
    elif case["kind"] == "halves":
        rho = min(rho, 0.75)
        nbytes, flops = _layer_work(R, K_in, K_out, e, rho, nu, R, 0.75 * R, rho * nu * R)
        nbytes += rho * R * K_in * e + 4 * R
    else:
        # the exact backward, and per draw one dW under each of the two masks; G, X and W once
        nbytes, flops = _layer_work(R, K_in, K_out, e, 1.0, 1.0, R, R, R)
        flops += 2.0 * R * K_in * K_out * case["M"] * (rho + rho * nu)
        nbytes += 16 * (K_in * K_out // 100)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Masks, counts and norms follow one written order of operations and are exact for given inputs ("differ" 0).
    # fp32 gradients: fp32 products and sums over up to 4096 terms in any order, about sqrt(4096) * 2^-24 = 4e-6.
    # bf16 gradients: fp32 sums, then dX rounded to bf16, and the scaled operand of dW rounded to bf16, either of
    # the two operands: 2^-9 / sqrt(3) = 1.1e-3 each, 2.3e-3 between two such results at the most; the largest
    # single difference is one rounding of a value, or of an operand against the root mean square of dW.
    if case["kind"] == "stack":
        # The dX of one layer is the G of the next.  Measured with every dX of the three listed stacks taken from an
        # fp32 product instead (sums in another order, 3e-5 to 6e-5 of dX): uniforms that lie between a token's two
        # keep probabilities flip 0 to 45 of 200 to 400 thousand token masks (up to 1.5e-4), and a flipped token is up to
        # 9 % of its own layer's dW, up to 2.5e-3 of all of dW; q moves by up to 8e-4.
        return {"rel": 1e-2, "max": 0.9, "differ": 6e-4}
    if case["dtype"] == F32:
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 1e-2, "max": 0.2}
