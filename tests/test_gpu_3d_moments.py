"""Moments and totals of large three-dimensional lattices, on both sides of the
sizes where they go from tiles to rows of nodes, against the oracle's relations
on the stored state (evaluated on the GPU in binary64)."""
import pytest
import torch

import workloads as wl
from oracle import qilbm_oracle3d as O
from test_gpu_3d import _co, _lattice, _problem

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float((a - b).abs().max() / b.abs().max())


# rows: layers of 200 000 nodes, of 36 000 from 4 million nodes on, or a quarter of
# the tiles' lanes idle; each with a lattice next to it that takes tiles
@pytest.mark.parametrize("nx,ny,nz,bc", [
    (512, 400, 10, wl.WALLS_Z), (512, 388, 10, wl.PERIODIC), (192, 190, 111, wl.WALLS_Z),
    (192, 190, 109, wl.PERIODIC), (1000, 650, 3, wl.WALLS_Z), (200, 110, 100, wl.WALLS_Z)])
def test_fp64_moments_match_oracle(nx, ny, nz, bc):
    """phi and rho to the order of 19 summands, mu, p and u as sums of at most 60
    terms, the largest 20 times the result: 1200 roundings, 1.4e-13."""
    print(f"case moments {nx}x{ny}x{nz} bc={bc}", flush=True)
    pb = _problem(nx, ny, nz, bc, (1e-6, -2e-6, -1e-5))
    f0, g0 = wl.random_state3d(nx, ny, nz, seed=nx + nz)
    lat = _lattice(pb, g0.sum(0))
    lat.set_state(f0, g0)
    m = O.macroscopic(*lat.get_state(), _co(pb))
    got = lat.moments()
    for k in ("phi", "rho"):
        assert _rel(got[k], m[k]) < 1e-14, k
    for k, ref in (("mu", m["mu"]), ("p", m["p"]), ("ux", m["u"][0]), ("uy", m["u"][1]),
                   ("uz", m["u"][2])):
        assert _rel(got[k], ref) < 1.4e-13, k
    assert torch.equal(lat.moments(("phi",))["phi"], got["phi"])


@pytest.mark.parametrize("precision,tol", [("fp64", (1e-14, 1e-12)), ("fp32", (1e-14, 2e-5))])
@pytest.mark.parametrize("nx,ny,nz,bc", [(150, 145, 114, wl.WALLS_Z), (150, 145, 116, wl.PERIODIC),
                                         (453, 452, 15, wl.WALLS_Z)])
def test_totals_match_oracle(nx, ny, nz, bc, precision, tol):
    """phi by rows from 2.5 million nodes and 16 layers on; bounds as on small
    lattices (momenta relative to the sum of their magnitudes)."""
    print(f"case totals {nx}x{ny}x{nz} bc={bc} {precision}", flush=True)
    pb = _problem(nx, ny, nz, bc, (1e-6, -2e-6, -1e-5))
    f0, g0 = wl.random_state3d(nx, ny, nz, seed=nx + nz)
    lat = _lattice(pb, g0.sum(0), precision)
    lat.set_state(f0, g0)
    m = O.macroscopic(*lat.get_state(), _co(pb))
    got = lat.mass()
    for a, ref in enumerate((m["phi"], m["rho"])):
        assert got[a] == pytest.approx(float(ref.sum()), rel=tol[0])
    for a in range(3):
        ru = m["rho"] * m["u"][a]
        assert abs(got[2 + a] - float(ru.sum())) <= tol[1] * float(ru.abs().sum())
