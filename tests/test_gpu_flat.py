"""Lattices of long rows, where the row sweeps take over from the tiles at
smaller sizes: on both sides of the change, forward against the oracle and
adjoint against the three kernels.

Tolerances (max |a - b| / max |b|): those of the other kernels from a random
state (forward, three steps: FP64 f 2e-11 and g 1e-12, FP32 3e-5 and 1e-6, FP16
storage 4e-3; adjoint FP64 1e-13, FP32 1e-5, parameter sums 1e-10 and 1e-3)."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import qilbm_oracle as O
from q229 import q229_total

pytestmark = pytest.mark.gpu

TOL = {"fp64": (2e-11, 1e-12), "fp32": (3e-5, 1e-6), "fp16": (4e-3, 4e-3)}
ADJ_TOL = {"fp64": (1e-13, 1e-10), "fp32": (1e-5, 1e-3)}


def _rel(a, b):
    return float((a.cpu() - b.cpu()).abs().max() / b.abs().max().clamp_min(1e-300))


@pytest.mark.parametrize("nx,ny,bc,precision", [
    (40009, 5, wl.WALLS_Y, "fp64"), (120011, 5, wl.PERIODIC, "fp64"),
    (22229, 9, wl.PERIODIC, "fp32"), (66673, 9, wl.WALLS_Y, "fp32"),
    (66673, 3, wl.WALLS_Y, "fp16"), (200017, 3, wl.PERIODIC, "fp16")])
def test_steps_match_oracle(nx, ny, bc, precision):
    from paper_1507_03521_amd import Lattice
    print(f"case flat {nx}x{ny} bc={bc} {precision}", flush=True)
    pb = wl.droplet64().with_(nx=nx, ny=ny, bc=bc, gx=2e-5, gy=-1e-5, rho_ref=0.3)
    f, g = wl.random_state(nx, ny, seed=nx)
    lat = Lattice(pb.as_dict(), np.full((ny, nx), 0.5), precision=precision, device="cuda:0")
    lat.set_state(f, g)
    ref = tuple(t.cpu() for t in lat.get_state())
    fixed = precision != "fp64"
    before = q229_total(lat.save_raw(), precision, nx, ny) if fixed else 0
    lat.step(3)
    with torch.no_grad():
        ref = O.run(None, O.coefficients_of(pb), 3, state=ref)
    got = lat.get_state()
    tf, tg = TOL[precision]
    assert _rel(got[0], ref[0]) < tf and _rel(got[1], ref[1]) < tg
    if fixed:
        assert q229_total(lat.save_raw(), precision, nx, ny) == before


@pytest.mark.parametrize("nx,ny,bc,precision", [
    (35311, 17, wl.WALLS_Y, "fp64"), (58831, 17, wl.PERIODIC, "fp64"),
    (22229, 9, wl.WALLS_Y, "fp32"), (66673, 9, wl.PERIODIC, "fp32")])
def test_adjoint_matches_three_kernels(nx, ny, bc, precision):
    from paper_1507_03521_amd import LBM_FLAG_UNFUSED, Lattice
    print(f"case flat adjoint {nx}x{ny} bc={bc} {precision}", flush=True)
    pb = wl.droplet64().with_(nx=nx, ny=ny, bc=bc, gx=1e-5, gy=-2e-5, rho_ref=0.5)
    f, g = wl.random_state(nx, ny, seed=nx)
    rng = np.random.default_rng(5)
    # cotangents of one sign, so that the parameter sums keep their digits
    fbar, gbar = rng.random((9, ny, nx)), rng.random((9, ny, nx))
    out, record = [], None
    for flags in (0, LBM_FLAG_UNFUSED):
        lat = Lattice(pb.as_dict(), np.full((ny, nx), 0.5), precision=precision, flags=flags,
                      device="cuda:0")
        if record is None:
            lat.set_state(f, g)
            record = lat.step_record()
        lat.adjoint_begin(torch.zeros((ny, nx), dtype=torch.float64, device="cuda:0"))
        lat.adjoint_set(fbar, gbar)
        lat.adjoint_step_record(record)
        lat.adjoint_step_record(record)
        out.append(lat.adjoint_get())
        lat.close()
    (f1, g1, s1, m1), (f3, g3, s3, m3) = out
    tol, ptol = ADJ_TOL[precision]
    assert _rel(f1, f3) <= tol and _rel(g1, g3) <= tol
    assert abs(s1 - s3) <= ptol * abs(s3) and abs(m1 - m3) <= ptol * abs(m3)
