"""The FP32 z-sweep step at the sizes that take it: from the lanes that tiles
would need on, against what a round of the sweep's workgroups takes (small
lattices run tiles, whatever their shape)."""
import pytest
import torch

import workloads as wl
from oracle import qilbm_oracle3d as O
from test_gpu_3d import FUSED_TOL, TOL, _lattice, _problem, _rel

pytestmark = pytest.mark.gpu


def _up(n, k):
    return (n + k - 1) // k


def takes_z_sweep(nx, ny, nz):
    """The rule of lbm3_step, on the 256 compute units of an MI355X."""
    tx = 16 if _up(nx, 16) * 64 <= _up(nx, 32) * 96 else 32
    lanes = _up(nx, tx) * tx * _up(ny, 4) * 4 * _up(nz, 4) * 4
    seg = _up(nz, min(nz, max(1, 256 // (_up(nx, 64) * _up(ny, 16)))))
    return lanes > 113000 * (seg + 6)


# one ragged column of tiles, one ragged row, one column more, segments of three
# planes and of one layer of the lattice, many ragged tiles
SHAPES = [(33, 1000, 33), (49, 400, 49), (257, 15, 300), (65, 31, 600), (97, 1000, 5),
          (2049, 129, 3), (129, 257, 33), (97, 97, 129)]


def _magic_lattice(pb, magic, phi0, flags=0, stream=None):
    from paper_1507_03521_amd import Lattice3D
    return Lattice3D(dict(pb.as_dict(), trt_magic=magic), phi0, precision="fp32", flags=flags,
                     device="cuda:0", stream=stream)


@pytest.mark.parametrize("bc", [wl.PERIODIC, wl.WALLS_Z])
@pytest.mark.parametrize("nx,ny,nz", SHAPES)
def test_z_sweep_matches_oracle_and_tiles(nx, ny, nz, bc):
    """One step against the oracle (on the GPU in binary64) from the stored
    state, two more against the tiles from the same state; the lattice total of
    phi exactly."""
    from paper_1507_03521_amd import LBM_FLAG_UNFUSED
    assert takes_z_sweep(nx, ny, nz)
    print(f"case z-sweep {nx}x{ny}x{nz} bc={bc}", flush=True)
    pb = _problem(nx, ny, nz, bc, (1e-6, -2e-6, -1e-5))
    magic = 0.25 if nx % 4 == 1 and bc else 0.0
    co = O.coefficients(pb.rho_A, pb.rho_B, pb.sigma, pb.W, pb.M, pb.tau_f, pb.tau_g,
                        pb.gx, pb.gy, pb.gz, pb.ref_density, pb.bc, trt_magic=magic)
    f0, g0 = wl.random_state3d(nx, ny, nz, seed=nz * 7 + nx)
    a = _magic_lattice(pb, magic, g0.sum(0))
    b = _magic_lattice(pb, magic, g0.sum(0), LBM_FLAG_UNFUSED)
    for lat in (a, b):
        lat.set_state(f0, g0)
    total = a.mass()[0]
    ref = O.step(*a.get_state(), co)
    a.step(1)
    got = a.get_state()
    assert _rel(got[0], ref[0]) < TOL["fp32"][0] and _rel(got[1], ref[1]) < TOL["fp32"][1]
    del ref, got
    a.step(2)
    b.step(3)
    (fa, ga), (fb, gb) = a.get_state(), b.get_state()
    tf, tg = FUSED_TOL["fp32"]
    assert _rel(fa, fb) < tf and _rel(ga, gb) < tg
    assert a.mass()[0] == b.mass()[0] == total


@pytest.mark.parametrize("nx,ny,nz,magic", [(129, 257, 33, 0.0), (97, 97, 129, 0.25)])
def test_state_replaced_between_sweeps(nx, ny, nz, magic):
    """The sweep keeps the next step's phi words from step to step: a state that
    replaces the stepped one is stepped with its own, in the bits of a lattice
    that never held another; and again after one step, two and three (either of
    its two buffers)."""
    assert takes_z_sweep(nx, ny, nz)
    pb = _problem(nx, ny, nz, wl.WALLS_Z, (1e-6, -2e-6, -1e-5))
    states = [wl.random_state3d(nx, ny, nz, seed=s) for s in (1, 2)]
    lat = _magic_lattice(pb, magic, states[0][1].sum(0))
    for k in (1, 2, 3):
        lat.set_state(*states[0])
        lat.step(k)
        lat.set_state(*states[1])
        lat.moments(("phi",))
        lat.step(2)
        other = _magic_lattice(pb, magic, states[1][1].sum(0))
        other.set_state(*states[1])
        other.step(2)
        assert all(torch.equal(x, y) for x, y in zip(lat.get_state(), other.get_state()))
        assert lat.mass() == other.mass()
        other.close()


def test_sweeps_captured_in_a_hip_graph():
    """Two steps captured and replayed three times, with eager work between, give
    the bits of eager stepping after every replay."""
    nx, ny, nz = 129, 257, 33
    assert takes_z_sweep(nx, ny, nz)
    pb = _problem(nx, ny, nz, wl.WALLS_Z, (0.0, 1e-6, -1e-5))
    f0, g0 = wl.random_state3d(nx, ny, nz, seed=9)
    s = torch.cuda.Stream()
    captured = _magic_lattice(pb, 0.0, g0.sum(0), stream=s)
    eager = _lattice(pb, g0.sum(0), "fp32")
    for lat in (captured, eager):
        lat.set_state(f0, g0)
        lat.step(1)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        captured.step(2)         # captured, not executed
    torch.cuda.synchronize()

    def same():
        a, b = captured.get_state(), eager.get_state()
        torch.cuda.synchronize()
        return torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])

    assert same()
    for _ in range(3):
        graph.replay()
        eager.step(2)
        torch.cuda.synchronize()
        captured.moments(("phi",))
        assert same()
