"""Records of steps on lattices near the largest tiled ones, where they are
stored as a stream."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


# both sides of the size (two buffers and a record, 190 MiB) from which on
# records are a stream: fp64 590 and 601 thousand nodes, fp32 1.17 and 1.2 million,
# fp16 1.96 and 2.0 million; and larger
@pytest.mark.parametrize("nx,ny,precision", [
    (769, 768, "fp64"), (771, 780, "fp64"), (889, 891, "fp64"), (1081, 1082, "fp32"),
    (1093, 1098, "fp32"), (1201, 1211, "fp32"), (1399, 1401, "fp16"), (1409, 1420, "fp16"),
    (1709, 1711, "fp16")])
def test_records_hold_the_moments_of_each_state(nx, ny, precision):
    """Four recorded steps end in the bits of four plain ones, and record k holds
    phi, mu and p of the state that step k started from: phi in FP64 to ten
    roundings of the state's moment, in the fixed-point formats exactly (the sum
    of the stored Q2.29 contributions, FP16 halves truncated to them); mu and p
    (FP64, FP32) as sums of at most 30 terms, the largest 20 times the result."""
    from paper_1507_03521_amd import Lattice
    print(f"case records {nx}x{ny} {precision}", flush=True)
    pb = wl.droplet64().with_(nx=nx, ny=ny, bc=wl.WALLS_Y, gx=2e-5, gy=-1e-5, rho_ref=0.3)
    f, g = wl.random_state(nx, ny, seed=nx)
    lats = [Lattice(pb.as_dict(), np.full((ny, nx), 0.5), precision=precision, device="cuda:0")
            for _ in range(2)]
    for lat in lats:
        lat.set_state(f, g)
    a, b = lats
    n, dt = 4, torch.float64 if precision == "fp64" else torch.float32
    recs = [torch.zeros(a.record_bytes, dtype=torch.uint8, device="cuda:0") for _ in range(n)]
    a.step_records(recs)
    ns = a.record_bytes // (6 * dt.itemsize)
    eps = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    for k in range(0, n, 2):
        # pairs of steps, so that the state between them is the recorded run's
        m = b.moments(("phi", "mu", "p"))
        rec = recs[k].view(dt).view(6, ns)[:, :nx * ny].view(6, ny, nx)
        if precision != "fp64":
            gs = b.get_state()[1]
            phi_q = (gs * 2.0 ** 29).trunc().sum(0)
            assert torch.equal(rec[0], phi_q.float() * 2.0 ** -29)
        for i, name in enumerate(("phi", "mu", "p")):
            if precision == "fp16" or (precision == "fp32" and i == 0):
                continue
            err = float((rec[i].double() - m[name]).abs().max() / m[name].abs().max())
            assert err <= (600 if i else 10) * eps, (k, name, err)
        b.step(2)
    assert torch.equal(a.save_raw(), b.save_raw())
