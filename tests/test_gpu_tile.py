"""Tiled step kernels of small and medium lattices, against the FP64 oracle.

The tile shape and the steps per launch go by the number of tiles (8 x 4,
16 x 4, 32 x 8 at two steps per launch; 16 x 4 or 16 x 8, then 32 x 4 or 32 x 8
at one), up to the lattices whose two population buffers fill 256 MiB. Sizes
here sit on both sides of each change of shape, on whole tiles and one node
off them, below the halo's width, and at the largest FP64 lattice of the range;
3 steps are a pair and a single step.

Tolerances (max |a - b| / max |b| per population set) are those of the other
forward kernels from a random state after a few steps: FP64 f 2e-11 and g
1e-12, FP32 3e-5 and 1e-6, FP16 storage 4e-3 for both.
"""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import qilbm_oracle as O
from q229 import q229_total

pytestmark = pytest.mark.gpu

TOL = {"fp64": (2e-11, 1e-12), "fp32": (3e-5, 1e-6), "fp16": (4e-3, 4e-3)}


def _rel(a, b):
    return float((a.cpu() - b).abs().max() / b.abs().max().clamp_min(1e-300))


@pytest.mark.parametrize("nx,ny,bc,precision", [
    (3, 3, wl.PERIODIC, "fp64"), (3, 3, wl.WALLS_Y, "fp32"), (3, 5, wl.WALLS_Y, "fp16"),
    (8, 4, wl.WALLS_Y, "fp64"), (9, 5, wl.WALLS_Y, "fp32"), (31, 9, wl.WALLS_Y, "fp16"),
    (64, 128, wl.PERIODIC, "fp64"), (65, 128, wl.WALLS_Y, "fp64"), (129, 64, wl.WALLS_Y, "fp32"),
    (128, 128, wl.WALLS_Y, "fp32"), (129, 128, wl.WALLS_Y, "fp64"), (128, 129, wl.PERIODIC, "fp32"),
    (128, 129, wl.WALLS_Y, "fp16"), (256, 256, wl.WALLS_Y, "fp64"), (257, 256, wl.WALLS_Y, "fp64"),
    (256, 257, wl.PERIODIC, "fp32"), (961, 967, wl.WALLS_Y, "fp64")])
def test_tiles_match_oracle(nx, ny, bc, precision):
    from paper_1507_03521_amd import Lattice
    print(f"case tiles {nx}x{ny} bc={bc} {precision}", flush=True)
    pb = wl.droplet64().with_(nx=nx, ny=ny, bc=bc, gx=2e-5, gy=-1e-5, rho_ref=0.3)
    f, g = wl.random_state(nx, ny, seed=nx * 7 + ny)
    lat = Lattice(pb.as_dict(), np.full((ny, nx), 0.5), precision=precision, device="cuda:0")
    lat.set_state(f, g)
    ref = tuple(t.cpu() for t in lat.get_state())          # the stored state
    fixed = precision != "fp64"
    before = q229_total(lat.save_raw(), precision, nx, ny) if fixed else 0
    n = 3
    lat.step(n)
    assert lat.time == n
    with torch.no_grad():
        ref = O.run(None, O.coefficients_of(pb), n, state=ref)
    got = lat.get_state()
    ef, eg = _rel(got[0], ref[0]), _rel(got[1], ref[1])
    print(f"  rel f {ef:.2e} g {eg:.2e}", flush=True)
    assert ef < TOL[precision][0] and eg < TOL[precision][1]
    if fixed:
        assert q229_total(lat.save_raw(), precision, nx, ny) == before


@pytest.mark.parametrize("nx,ny,bc,precision", [
    (3, 3, wl.WALLS_Y, "fp64"), (17, 9, wl.PERIODIC, "fp32"), (31, 7, wl.WALLS_Y, "fp16"),
    (511, 511, wl.WALLS_Y, "fp64"), (513, 500, wl.WALLS_Y, "fp64"), (577, 479, wl.PERIODIC, "fp32"),
    (640, 497, wl.WALLS_Y, "fp32"), (515, 523, wl.WALLS_Y, "fp16")])
def test_moments_and_totals_match_oracle(nx, ny, bc, precision):
    """16 x 8 tiles of the moments on small lattices, 64 x 8 and (FP32) 64 x 16
    from 512 tiles on, and totals of 32 x 8 tiles shared out over workgroups:
    the moments of the state that the GPU holds. phi is one rounding of an
    exact sum, rho two more. mu, u and p are sums of at most 30 terms, the
    largest 20 times the result (a Laplacian of mu, itself one of phi): 30 x 20
    roundings of the compute type, 7e-14 and 4e-5."""
    from paper_1507_03521_amd import Lattice
    print(f"case moments {nx}x{ny} bc={bc} {precision}", flush=True)
    pb = wl.droplet64().with_(nx=nx, ny=ny, bc=bc, gx=2e-5, gy=-1e-5, rho_ref=0.3)
    f, g = wl.random_state(nx, ny, seed=nx + 3 * ny)
    lat = Lattice(pb.as_dict(), np.full((ny, nx), 0.5), precision=precision, device="cuda:0")
    lat.set_state(f, g)
    fs, gs = (t.cpu() for t in lat.get_state())
    co = O.coefficients_of(pb)
    ref = dict(zip(("phi", "rho", "ux", "uy", "p", "mu"), O.moments(fs, gs, co)))
    got = lat.moments()
    fp64 = precision == "fp64"
    eps = 2.0 ** -24
    tol = dict(phi=1e-14 if fp64 else 2 * eps, rho=1e-14 if fp64 else 4 * eps,
               **dict.fromkeys(("mu", "p", "ux", "uy"), 7e-14 if fp64 else 4e-5))
    for k, r in ref.items():
        assert _rel(got[k], r) < tol[k], k
    assert torch.equal(lat.moments(("phi",))["phi"], got["phi"])
    t = lat.mass()
    if precision == "fp16":
        return                   # the totals take binary16 g as Q2.29 contributions
    rho, n = ref["rho"], nx * ny
    exact = (float(ref["phi"].sum()), float(rho.sum()), float((rho * ref["ux"]).sum()),
             float((rho * ref["uy"]).sum()))
    scale = (n, n, float((rho * ref["ux"]).abs().sum()), float((rho * ref["uy"]).abs().sum()))
    for a, b, s, w in zip(t, exact, scale, (1e-14, 1e-14, tol["ux"], tol["uy"])):
        assert abs(a - b) <= w * s
