"""Moments of the stored state: what each storage format may lose."""
import numpy as np
import pytest
import torch

import workloads as wl

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
