"""The row-sweeping adjoint, which only lattices beyond the tiled ones take
(two cotangent buffers and a record of more than 325 MiB in FP64, 256 MiB in
FP32), against the three kernels (LBM_FLAG_UNFUSED) on the same record.

Near-square lattices with walls and periodic, lattices narrower than the halo,
of one strip and one column more, of ragged strips, and of fewer rows than a
segment has. Tolerances (max |a - b| / max |b|): FP64 1e-13 and FP32 1e-5 for the
cotangents, 1e-10 and 1e-3 for the parameter sums."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

TOL = {"fp64": (1e-13, 1e-10), "fp32": (1e-5, 1e-3)}


@pytest.mark.parametrize("nx,ny,bc,precision", [
    (1301, 1307, wl.WALLS_Y, "fp32"), (1303, 1301, wl.PERIODIC, "fp32"),
    (3, 540007, wl.WALLS_Y, "fp32"), (7, 230003, wl.PERIODIC, "fp32"),
    (248, 6503, wl.WALLS_Y, "fp32"), (249, 6473, wl.PERIODIC, "fp32"),
    (523, 3089, wl.WALLS_Y, "fp32"), (540011, 3, wl.WALLS_Y, "fp32"),
    (90001, 18, wl.PERIODIC, "fp32"),
    (3, 341003, wl.PERIODIC, "fp64"), (16, 64007, wl.WALLS_Y, "fp64"),
    (249, 4111, wl.WALLS_Y, "fp64"), (523, 1951, wl.PERIODIC, "fp64"),
    (60013, 17, wl.WALLS_Y, "fp64")])
def test_row_sweep_matches_three_kernels(nx, ny, bc, precision):
    from paper_1507_03521_amd import LBM_FLAG_UNFUSED, Lattice
    print(f"case adjoint sweep {nx}x{ny} bc={bc} {precision}", flush=True)
    size = 8 if precision == "fp64" else 4
    assert 42 * nx * ny * size > (325 if precision == "fp64" else 256) << 20
    pb = wl.droplet64().with_(nx=nx, ny=ny, bc=bc, gx=1e-5, gy=-2e-5, rho_ref=0.5)
    dev = torch.device("cuda:0")
    f, g = wl.random_state(nx, ny, seed=nx + ny)
    gen = torch.Generator(device=dev).manual_seed(5)
    # cotangents of one sign, so that the parameter sums keep their digits
    fbar, gbar = (torch.rand((9, ny, nx), generator=gen, device=dev, dtype=torch.float64)
                  for _ in range(2))
    out, record = [], None
    for flags in (0, LBM_FLAG_UNFUSED):
        lat = Lattice(pb.as_dict(), np.full((ny, nx), 0.5), precision=precision, flags=flags,
                      device=dev)
        if record is None:
            lat.set_state(f, g)
            record = lat.step_record()
        lat.adjoint_begin(torch.zeros((ny, nx), dtype=torch.float64, device=dev))
        for _ in range(2):                       # the second must start from cleared sums
            lat.adjoint_set(fbar, gbar)
            lat.adjoint_step_record(record)
            lat.adjoint_step_record(record)
        out.append(lat.adjoint_get())
        lat.close()
    (f1, g1, s1, m1), (f3, g3, s3, m3) = out
    tol, ptol = TOL[precision]
    ef = float((f1 - f3).abs().max() / f3.abs().max())
    eg = float((g1 - g3).abs().max() / g3.abs().max())
    es, em = abs(s1 - s3) / abs(s3), abs(m1 - m3) / abs(m3)
    print(f"  rel f {ef:.2e} g {eg:.2e} sigma {es:.2e} M {em:.2e}", flush=True)
    assert ef <= tol and eg <= tol and es <= ptol and em <= ptol
