"""Helpers shared by the GPU parity tests, the smoke check and the benchmark:
move seeded inputs to the device, run the library, bring results back."""
from __future__ import annotations

import numpy as np
import torch

import workloads
from paper_2402_17227_amd import binding as vb


to_device = vb.to_device     # numpy (fp32, or bf16 bit patterns as uint16) -> device tensor of the layer dtype


def from_device(t: torch.Tensor) -> np.ndarray:
    """device tensor -> numpy float64 (values) for comparison."""
    return t.detach().float().cpu().numpy().astype(np.float64)


def rel_l2(got, ref) -> float:
    got = np.asarray(got, np.float64)
    ref = np.asarray(ref, np.float64)
    den = float(np.sqrt((ref**2).sum()))
    num = float(np.sqrt(((got - ref) ** 2).sum()))
    return num / den if den > 0 else num


def rel_l2_rows(got, ref) -> float:
    """Worst relative L2 error of a single row (dX: every row carries its own sample's and token's scale, so
    a row is the natural unit).  A bound on every row implies the same bound on the whole tensor, and a
    misplaced or stale tile cannot hide behind the rows with the large norms.  Rows that are zero in the
    reference (dropped samples) must be exactly zero."""
    got = np.asarray(got, np.float64).reshape(np.shape(ref))
    ref = np.asarray(ref, np.float64)
    if ref.size == 0:
        return 0.0
    num = np.sqrt(((got - ref) ** 2).sum(axis=-1))
    den = np.sqrt((ref ** 2).sum(axis=-1))
    zero = den == 0
    if np.any(num[zero] != 0):
        return float("inf")
    return float((num[~zero] / den[~zero]).max()) if np.any(~zero) else 0.0


def rel_l2_tiles(got, ref, tile: int = 128) -> float:
    """Worst relative L2 error of a tile x tile block of a matrix (dW: one block = one workgroup's output
    tile of the largest weight-gradient kernel, and a multiple of the smaller kernels' tiles); implies the
    same bound on the whole matrix."""
    got = np.asarray(got, np.float64).reshape(np.shape(ref))
    ref = np.asarray(ref, np.float64)
    worst = 0.0
    for r0 in range(0, ref.shape[0], tile):
        for c0 in range(0, ref.shape[1], tile):
            worst = max(worst, rel_l2(got[r0:r0 + tile, c0:c0 + tile], ref[r0:r0 + tile, c0:c0 + tile]))
    return worst


def run_layer_gpu(spec, G, X, W, draw: int = 0, token_sampling: bool = True, want_dX=True, want_dW=True):
    """One call of vcas_linear_backward.  Returns (plan as numpy dict, dX fp64, dW fp64)."""
    shape = vb.shape_of(spec.N, spec.T, spec.K_in, spec.K_out, spec.dtype)
    g, x, w = to_device(G, spec.dtype), to_device(X, spec.dtype), to_device(W, spec.dtype)
    plan = vb.Plan.allocate(spec.N, spec.T)
    ws = vb.make_workspace(shape)
    dX = torch.full((spec.R, spec.K_in), float("nan"), dtype=g.dtype, device="cuda") if want_dX else None
    dW = torch.full((spec.K_out, spec.K_in), float("nan"), dtype=torch.float32, device="cuda") if want_dW else None
    rng = vb.Rng(spec.seed, spec.layer, draw)
    vb.vcas_linear_backward(shape, g, x, w, spec.rho, spec.nu, rng, token_sampling, plan, dX, dW, ws)
    torch.cuda.synchronize()
    return plan_to_numpy(plan), (from_device(dX) if want_dX else None), (from_device(dW) if want_dW else None)


def plan_to_numpy(plan: "vb.Plan") -> dict:
    d = {k: getattr(plan, k).cpu().numpy() for k in ("gsq", "gnorm", "p", "maskA", "xsq", "score", "q", "maskW", "scaleW")}
    cntA = int(plan.cntA.item())
    cntW = int(plan.cntW.item())
    d["cntA"], d["cntW"] = cntA, cntW
    d["idxA"] = plan.idxA.cpu().numpy()[:cntA]
    d["idxW"] = plan.idxW.cpu().numpy()[:cntW]
    return d


def compare_plan(got: dict, want) -> None:
    """Bit-exact comparison of every sampling decision with the oracle's plan."""
    for name in ("gsq", "gnorm", "p", "xsq", "score", "q", "scaleW"):
        a, b = got[name], getattr(want, name)
        assert a.dtype == np.float32 and b.dtype == np.float32
        same = a.view(np.uint32) == b.view(np.uint32)
        assert same.all(), f"{name}: {int((~same).sum())} of {a.size} differ, first at {int(np.argmin(same))}: " \
                           f"{a[np.argmin(same)]!r} vs {b[np.argmin(same)]!r}"
    for name in ("maskA", "maskW"):
        assert np.array_equal(got[name], getattr(want, name)), name
    assert got["cntA"] == want.idxA.size and got["cntW"] == want.idxW.size
    assert np.array_equal(got["idxA"], want.idxA) and np.array_equal(got["idxW"], want.idxW)


def blocks_to_device_layout(blocks, fill=np.nan):
    """[R, nb] block sums (the oracle's) -> the library's layout [ceil(nb/4), R, 4]: four neighbouring blocks of
    a row side by side; the unused slots of the last group get `fill` (nobody may read them)."""
    R, nb = blocks.shape
    out = np.full(((nb + 3) // 4, R, 4), fill, np.float32)
    for b in range(nb):
        out[b // 4, :, b % 4] = blocks[:, b]
    return out


def blocks_from_device_layout(dev, nb):
    """The inverse: [groups, R, 4] -> [R, nb]."""
    a = dev.cpu().numpy() if hasattr(dev, "cpu") else np.asarray(dev)
    return np.stack([a[b // 4, :, b % 4] for b in range(nb)], axis=1)


def packs_the_kept_rows(ws, run, plan_only) -> bool:
    """Which form of the bf16 weight gradient run() takes, from what it leaves in the workspace: the packed form's operand lies behind
    everything that plan_only() (the same call without dW) writes, the partial tiles of either form lie in front of it."""
    def end(call):
        ws[8192:] = 0x5A      # all but the control words
        call()
        torch.cuda.synchronize()
        return int((ws != 0x5A).nonzero()[-1])
    without = end(plan_only)
    return end(run) > without
