"""Gradients of whole runs: step counts at the ends of their range."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nsteps", [0, -3])
def test_run_of_no_steps_is_the_identity(nsteps, precision):
    """No steps (a count below zero is none): phi = phi0, to the rounding of
    its nine summands, and its gradient the weight, no part of it from sigma
    and M, whose terms cancel in the sum."""
    from paper_1507_03521_amd.autograd import simulate
    pb = wl.droplet64().with_(nx=40, ny=33)
    rng = np.random.default_rng(3)
    dev = torch.device("cuda:0")
    phi0 = torch.tensor(rng.random((33, 40)), device=dev, requires_grad=True)
    sigma = torch.tensor(0.01, dtype=torch.float64, requires_grad=True)
    M = torch.tensor(0.1, dtype=torch.float64, requires_grad=True)
    weight = torch.tensor(rng.random((33, 40)), device=dev)
    phi = simulate(phi0, sigma, M, pb.as_dict(), nsteps, checkpoint=4, precision=precision)
    d0, ds, dm = torch.autograd.grad(phi, (phi0, sigma, M), weight)
    # fp64: a few roundings of values of order one; fp32: Q2.29 words, 2^-30
    # each, and binary32 sums and cotangents
    fp64 = precision == "fp64"
    assert float((phi.detach() - phi0.detach()).abs().max()) <= \
        (1e-14 if fp64 else 9 * 2.0 ** -30 + 2.0 ** -24)
    assert float((d0 - weight).abs().max()) <= (1e-14 if fp64 else 2.0 ** -24)
    # 1320 nodes of 1e-16 (binary64 sums of the same nine cotangents) times
    # at most 0.2 / sigma and 0.2 / M
    assert abs(float(ds)) <= 1e-11 and abs(float(dm)) <= 1e-11
