"""The tiled three-dimensional kernels at the sizes where one form hands over
to the next: one launch a step (up to 256 tiles of 4 x 4 x 4), two (256, in
FP32 512, of 8 x 4 x 4), three with tiles 16 or 32 wide, and the FP32 z-sweep
of large lattices."""
import pytest

import workloads as wl
from oracle import qilbm_oracle3d as O
from test_gpu_3d import FUSED_TOL, TOL, _problem, _rel

pytestmark = pytest.mark.gpu

def _lattice(pb, magic, phi0, precision, flags=0):
    from paper_1507_03521_amd import Lattice3D
    return Lattice3D(dict(pb.as_dict(), trt_magic=magic), phi0, precision=precision, flags=flags,
                     device="cuda:0")


SIZES = [(5, 4, 1021), (16, 16, 64), (15, 17, 63),            # one launch: 1 x 1 x 256 tiles, 256, 320
         (32, 32, 32), (33, 31, 30), (30, 61, 33), (57, 33, 25),  # two: 256 tiles, 320, 2 x that
         (33, 33, 40), (48, 37, 39), (49, 38, 35), (65, 34, 33)]  # three: 16 wide to 48, then 32


@pytest.mark.parametrize("bc", [wl.PERIODIC, wl.WALLS_Z])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny,nz", SIZES)
def test_two_steps_match_oracle(nx, ny, nz, precision, bc):
    pb = _problem(nx, ny, nz, bc, (1e-6, -2e-6, -1e-5))
    magic = 0.25 if (nx + ny) % 2 else 0.0
    co = O.coefficients(pb.rho_A, pb.rho_B, pb.sigma, pb.W, pb.M, pb.tau_f, pb.tau_g,
                        pb.gx, pb.gy, pb.gz, pb.ref_density, pb.bc, trt_magic=magic)
    f0, g0 = wl.random_state3d(nx, ny, nz, seed=nx + 7 * nz)
    lat = _lattice(pb, magic, g0.sum(0), precision)
    lat.set_state(f0, g0)
    f, g = (t.cpu() for t in lat.get_state())
    tf, tg = TOL[precision]
    for _ in range(2):
        # each step from the state that the GPU holds
        lat.step(1)
        f1, g1 = (t.cpu() for t in lat.get_state())
        fr, gr = O.step(f, g, co)
        assert _rel(f1, fr) < tf and _rel(g1, gr) < tg
        f, g = f1, g1


@pytest.mark.parametrize("nx,ny,nz,bc,trt", [(250, 250, 50, wl.WALLS_Z, 0.0),
                                             (256, 249, 51, wl.PERIODIC, 0.25)])
def test_z_sweep_of_large_lattices_matches_tiles(nx, ny, nz, bc, trt):
    pb = _problem(nx, ny, nz, bc, (1e-6, -2e-6, -1e-5))
    from paper_1507_03521_amd import LBM_FLAG_UNFUSED
    f0, g0 = wl.random_state3d(nx, ny, nz, seed=3)
    a = _lattice(pb, trt, g0.sum(0), "fp32")
    b = _lattice(pb, trt, g0.sum(0), "fp32", flags=LBM_FLAG_UNFUSED)
    for lat in (a, b):
        lat.set_state(f0, g0)
        lat.step(3)
    (fa, ga), (fb, gb) = a.get_state(), b.get_state()
    tf, tg = FUSED_TOL["fp32"]
    assert _rel(fa, fb) < tf and _rel(ga, gb) < tg
    assert a.mass()[0] == b.mass()[0]
