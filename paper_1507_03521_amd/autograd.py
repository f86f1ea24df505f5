"""Gradients of a final-time loss through the GPU lattice: a
``torch.autograd.Function`` whose backward runs the library's hand-written
adjoint step with checkpoint-and-recompute."""
from __future__ import annotations

import torch

from .lattice import Lattice


def _records(lat: Lattice, count: int) -> list:
    """count step records; small ones share one allocation."""
    nbytes = lat.record_bytes
    if count * nbytes <= 64 << 20:
        return list(torch.empty((count, nbytes), dtype=torch.uint8, device=lat.device))
    return [torch.empty(nbytes, dtype=torch.uint8, device=lat.device) for _ in range(count)]


class PhaseFieldRun(torch.autograd.Function):
    """phi_K = run(phi0; sigma, M) for K steps. Differentiable in phi0,
    sigma and M.

    Forward keeps a raw snapshot of the state every ``checkpoint`` steps
    (including t = 0) and advances each segment with one library call, which
    reads the segment's snapshot and writes the next one directly.
    Backward walks the segments last to first: it replays the segment from its
    snapshot with one call that also writes the records (the forward quantities
    phi, mu, p, S, j each adjoint step needs) -- the same launches as the
    forward segment, pairs of steps included -- and applies the adjoint step to
    the records in reverse time order, in one call. Memory:
    ceil(K / C) raw states plus C records (a record is a third of a raw
    state). With two steps per kernel pass, an even C keeps the launches of
    a run without checkpoints (pairs from even t), so the gradients do not
    depend on C bitwise; an odd C moves the pairs and changes only rounding.
    """

    @staticmethod
    def forward(ctx, phi0, sigma, M, params: dict, nsteps: int, checkpoint: int,
                precision: str = "fp64", flags: int = 0):
        p = dict(params)
        p["sigma"] = float(sigma)
        p["M"] = float(M)
        lat = Lattice(p, phi0.detach(), precision=precision, flags=flags, device=phi0.device)
        C, K = max(1, int(checkpoint)), int(nsteps)
        snaps = [lat.save_raw()] if K > 0 else []
        for t0 in range(0, K, C):
            dst = lat.empty_raw() if t0 + C < K else None
            lat.segment(min(C, K - t0), snaps[-1] if t0 else None, t0, dst=dst)
            if dst is not None:
                snaps.append(dst)
        phi = lat.moments(("phi",))["phi"]
        ctx.lat = lat
        ctx.param_meta = [(x.device, x.dtype) if torch.is_tensor(x) else None for x in (sigma, M)]
        ctx.snaps = snaps
        ctx.C = C
        ctx.K = K
        ctx.save_for_backward(phi0.detach())
        return phi

    @staticmethod
    def backward(ctx, dphi):
        (phi0,) = ctx.saved_tensors
        lat, snaps, C, K = ctx.lat, ctx.snaps, ctx.C, ctx.K
        lat.adjoint_begin(dphi.detach().to(torch.float64).contiguous())
        held = _records(lat, max(0, min(C, K)))
        records = lat.record_array(held)
        for s in reversed(range(len(snaps))):
            n = min(C, K - s * C)
            lat.segment(n, snaps[s], s * C, records=records)
            lat.adjoint_step_records(records, n)
        dphi0, dsigma, dM = lat.adjoint_init(phi0)
        grads = []
        for val, meta in zip((dsigma, dM), ctx.param_meta):
            grads.append(None if meta is None else torch.tensor(val, dtype=meta[1], device=meta[0]))
        return (dphi0.to(phi0.dtype), grads[0], grads[1], None, None, None, None, None)


def simulate(phi0: torch.Tensor, sigma: torch.Tensor, M: torch.Tensor, params: dict,
             nsteps: int, checkpoint: int = 100, precision: str = "fp64",
             flags: int = 0) -> torch.Tensor:
    """Order parameter after ``nsteps`` steps from ``phi0``; differentiable
    with respect to phi0, sigma and M (0-d tensors)."""
    return PhaseFieldRun.apply(phi0, sigma, M, params, nsteps, checkpoint, precision, flags)
