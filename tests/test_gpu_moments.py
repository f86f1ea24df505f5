"""Moments of the stored state: what each storage format may lose."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import qilbm_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,bc", [(3, 3, wl.PERIODIC), (33, 20, wl.WALLS_Y),
                                      (600, 520, wl.WALLS_Y)])
def test_fp16_phi_is_the_rounded_sum_of_the_halves(nx, ny, bc):
    """phi, alone and with the other fields, is the exact sum of the stored
    values rounded once to binary32: half a unit in the last place, 2^-24 of
    the value itself. Small phi, where a half has digits far below 2^-29."""
    from paper_1507_03521_amd import Lattice
    print(f"case fp16 phi {nx}x{ny} bc={bc}", flush=True)
    pb = wl.droplet64().with_(nx=nx, ny=ny, bc=bc, gx=2e-5, gy=-1e-5, rho_ref=0.3)
    f, g = wl.random_state(nx, ny, seed=nx + ny)
    lat = Lattice(pb.as_dict(), np.full((ny, nx), 0.5), precision="fp16", device="cuda:0")
    lat.set_state(f, 1e-4 * g)
    exact = lat.get_state()[1].sum(0)         # exact in binary64
    for names in (("phi",), ("phi", "rho", "ux", "uy", "p", "mu")):
        phi = lat.moments(names)["phi"]
        assert bool(((phi - exact).abs() <= 2.0 ** -24 * exact.abs()).all())


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("nx,ny,bc", [(3, 20011, wl.WALLS_Y), (10, 18760, wl.PERIODIC),
                                      (11, 18760, wl.WALLS_Y), (18, 18760, wl.WALLS_Y),
                                      (19, 18760, wl.PERIODIC), (20003, 3, wl.WALLS_Y)])
def test_moments_and_totals_of_thin_lattices(nx, ny, bc, precision):
    """Lattices of few columns, on both sides of the widths where the moments
    (18 and 19) and the totals (10 and 11) go from a node per thread to tiles,
    against the oracle on the stored state. Bounds as on other lattices: phi
    one rounding, rho two more, the others 600 roundings of the compute type;
    the totals those of their summands."""
    from paper_1507_03521_amd import Lattice
    from paper_1507_03521_amd.lattice import mass_noalloc
    print(f"case thin moments {nx}x{ny} bc={bc} {precision}", flush=True)
    pb = wl.droplet64().with_(nx=nx, ny=ny, bc=bc, gx=2e-5, gy=-1e-5, rho_ref=0.3)
    f, g = wl.random_state(nx, ny, seed=nx + 3 * ny)
    lat = Lattice(pb.as_dict(), np.full((ny, nx), 0.5), precision=precision, device="cuda:0")
    lat.set_state(f, g)
    fs, gs = (t.cpu() for t in lat.get_state())
    ref = dict(zip(("phi", "rho", "ux", "uy", "p", "mu"),
                   O.moments(fs, gs, O.coefficients_of(pb))))
    got = lat.moments()
    fp64 = precision == "fp64"
    eps = 2.0 ** -24
    tol = dict(phi=1e-14 if fp64 else 2 * eps, rho=1e-14 if fp64 else 4 * eps,
               **dict.fromkeys(("mu", "p", "ux", "uy"), 7e-14 if fp64 else 4e-5))
    for k, r in ref.items():
        assert float((got[k].cpu() - r).abs().max() / r.abs().max()) < tol[k], k
    assert torch.equal(lat.moments(("phi",))["phi"], got["phi"])
    t = lat.mass()
    out = torch.empty(4, dtype=torch.float64, device="cuda:0")
    mass_noalloc(pb.as_dict(), precision, lat.save_raw(), out)
    assert tuple(out.tolist()) == t
    if precision == "fp16":
        return                   # the totals take binary16 g as Q2.29 contributions
    rho, n = ref["rho"], nx * ny
    exact = (float(ref["phi"].sum()), float(rho.sum()), float((rho * ref["ux"]).sum()),
             float((rho * ref["uy"]).sum()))
    scale = (n, n, float((rho * ref["ux"]).abs().sum()), float((rho * ref["uy"]).abs().sum()))
    for a, b, s, w in zip(t, exact, scale, (1e-14, 1e-14, tol["ux"], tol["uy"])):
        assert abs(a - b) <= w * s
