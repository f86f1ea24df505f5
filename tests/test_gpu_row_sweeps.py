"""The row-sweeping forward kernels where small lattices run tiles by
themselves: a number of rows per segment (set_pass, set_launch) selects them.

Lattices narrower than the halo, of one strip and of several with ragged tails,
and segments from one row to the whole lattice, in every storage type, against
the oracle. Tolerances (max |a - b| / max |b| per population set) from a random
state after a few steps, as for the other forward kernels: FP64 f 2e-11 and g
1e-12, FP32 3e-5 and 1e-6, FP16 storage 4e-3 for both; records FP64 1e-12, FP32
1e-4, FP16 storage 2e-3 of each field's largest magnitude.
"""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import qilbm_oracle as O
from q229 import q229_total

pytestmark = pytest.mark.gpu

TOL = {"fp64": (2e-11, 1e-12), "fp32": (3e-5, 1e-6), "fp16": (4e-3, 4e-3)}
REC_TOL = {"fp64": 1e-12, "fp32": 1e-4, "fp16": 2e-3}

SHAPES = [(37, 29, wl.PERIODIC, 0.0), (300, 70, wl.WALLS_Y, -1e-5), (520, 45, wl.PERIODIC, 0.0),
          (485, 33, wl.WALLS_Y, -2e-5), (3, 3, wl.PERIODIC, 0.0), (5, 4, wl.WALLS_Y, -1e-5),
          (10, 40, wl.PERIODIC, 0.0), (243, 12, wl.WALLS_Y, -1e-5)]


def _rel(a, b):
    return float((a.cpu() - b.cpu()).abs().max() / b.cpu().abs().max().clamp_min(1e-300))


def _lattice(pb, precision, per, seg_rows, magic=0.0):
    from paper_1507_03521_amd import Lattice
    lat = Lattice(dict(pb.as_dict(), trt_magic=magic), np.full((pb.ny, pb.nx), 0.5),
                  precision=precision, device="cuda:0")
    lat.set_pass(per, seg_rows if per == 2 else 0)
    lat.set_launch(seg_rows)       # single steps, also the last of an odd count
    info = lat.pass_info()
    assert info["steps"] == per and info["seg_rows"] == min(seg_rows, pb.ny)
    return lat


def _check_steps(pb, precision, per, seg_rows, n, magic=0.0):
    f, g = wl.random_state(pb.nx, pb.ny, seed=pb.nx + 7 * pb.ny)
    lat = _lattice(pb, precision, per, seg_rows, magic)
    lat.set_state(f, g)
    ref = tuple(t.cpu() for t in lat.get_state())
    fixed = precision != "fp64"
    before = q229_total(lat.save_raw(), precision, pb.nx, pb.ny) if fixed else 0
    lat.step(n)
    assert lat.time == n
    with torch.no_grad():
        ref = O.run(None, O.coefficients_of(pb, trt_magic=magic), n, state=ref)
    got = lat.get_state()
    ef, eg = _rel(got[0], ref[0]), _rel(got[1], ref[1])
    print(f"  rel f {ef:.2e} g {eg:.2e}", flush=True)
    assert ef < TOL[precision][0] and eg < TOL[precision][1]
    if fixed:
        assert q229_total(lat.save_raw(), precision, pb.nx, pb.ny) == before


@pytest.mark.parametrize("per", [1, 2])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("nx,ny,bc,gy", SHAPES)
def test_sweeps_match_oracle(nx, ny, bc, gy, precision, per):
    print(f"case sweep {precision} {nx}x{ny} bc={bc} per={per}", flush=True)
    pb = wl.droplet64().with_(nx=nx, ny=ny, bc=bc, gy=gy, rho_ref=0.55)
    _check_steps(pb, precision, per, 16, 5)


@pytest.mark.parametrize("seg_rows", [1, 2, 5, 8, 17, 1000])
@pytest.mark.parametrize("precision,per", [("fp64", 1), ("fp64", 2), ("fp32", 2), ("fp16", 1),
                                           ("fp16", 2)])
def test_segment_lengths(precision, per, seg_rows):
    print(f"case sweep {precision} per={per} seg_rows={seg_rows}", flush=True)
    pb = wl.droplet64().with_(nx=300, ny=41, bc=wl.WALLS_Y, gy=-1e-5, rho_ref=0.55)
    _check_steps(pb, precision, per, seg_rows, 4)


@pytest.mark.parametrize("magic", [3.0 / 16.0, 0.25])
@pytest.mark.parametrize("precision,per", [("fp64", 1), ("fp64", 2), ("fp32", 1), ("fp32", 2),
                                           ("fp16", 1), ("fp16", 2)])
@pytest.mark.parametrize("nx,ny,bc,gy", [SHAPES[0], SHAPES[1], SHAPES[5]])
def test_trt_sweeps_match_oracle(nx, ny, bc, gy, precision, per, magic):
    print(f"case trt sweep {precision} {nx}x{ny} per={per} magic={magic}", flush=True)
    pb = wl.droplet64().with_(nx=nx, ny=ny, bc=bc, gy=gy, rho_ref=0.55, tau_f=0.7)
    _check_steps(pb, precision, per, 9, 3, magic)


@pytest.mark.parametrize("seg_rows", [3, 16])
@pytest.mark.parametrize("precision,per", [("fp64", 1), ("fp64", 2), ("fp32", 1), ("fp32", 2),
                                           ("fp16", 1), ("fp16", 2)])
def test_sweep_records_match_steps_and_oracle(precision, per, seg_rows):
    """Recorded steps leave the bits of plain ones; record k holds the oracle's
    forward quantities after k steps."""
    nx, ny, n = 300, 41, 5
    pb = wl.droplet64().with_(nx=nx, ny=ny, bc=wl.WALLS_Y, gy=-1e-5, rho_ref=0.5)
    f, g = wl.random_state(nx, ny, seed=18)
    a, b = (_lattice(pb, precision, per, seg_rows) for _ in range(2))
    for lat in (a, b):
        lat.set_state(f, g)
    state = tuple(t.cpu() for t in a.get_state())
    recs = [torch.empty(a.record_bytes, dtype=torch.uint8, device="cuda:0") for _ in range(n)]
    a.step_records(recs)
    b.step(n)
    assert torch.equal(a.save_raw(), b.save_raw())
    dt = torch.float64 if precision == "fp64" else torch.float32
    co = O.coefficients_of(pb)
    for k in range(n):
        planes = recs[k].view(dt).view(6, -1)[:, :nx * ny].double().cpu().view(6, ny, nx)
        m = O.macroscopic(*state, co)
        for j, name in enumerate(("phi", "mu", "p", "S", "jx", "jy")):
            assert _rel(planes[j], m[name]) <= REC_TOL[precision], (k, name)
        with torch.no_grad():
            state = O.step(*state, co)


# no smaller lattice takes these by itself: FP64 above 220 MiB of populations, FP32
# above 224
@pytest.mark.parametrize("n", [1, 2, 5])
@pytest.mark.parametrize("nx,ny,precision,mib", [(1000, 900, "fp64", 220), (1403, 1300, "fp32", 224)])
def test_sweeps_from_and_into_snapshots(nx, ny, precision, mib, n):
    """A segment that sweeps rows from one snapshot into another gives the bits
    of the steps between copies."""
    from paper_1507_03521_amd import Lattice
    print(f"case sweep segment {nx}x{ny} {precision} n={n}", flush=True)
    pb = wl.droplet64().with_(nx=nx, ny=ny, bc=wl.WALLS_Y, gy=-1e-5, rho_ref=0.3)
    f, g = wl.random_state(nx, ny, seed=1)
    a, b = (Lattice(pb.as_dict(), np.full((ny, nx), 0.5), precision=precision, device="cuda:0")
            for _ in range(2))
    assert 2 * a.state_bytes > mib << 20
    a.set_state(f, g)
    s0, s1 = a.save_raw(), torch.zeros(a.state_bytes, dtype=torch.uint8, device="cuda:0")
    b.segment(n, src=s0, t=0, dst=s1)
    a.step(n)
    assert torch.equal(a.save_raw(), s1)


# the one-step tiles whose stores are written back: more than 600 000 nodes with nx a
# multiple of 16, 300 000 without; up to the largest of each type
@pytest.mark.parametrize("nx,ny,bc,precision", [
    (557, 541, wl.WALLS_Y, "fp64"), (800, 757, wl.PERIODIC, "fp64"), (893, 891, wl.WALLS_Y, "fp64"),
    (701, 433, wl.PERIODIC, "fp32"), (1024, 601, wl.WALLS_Y, "fp32"),
    (1261, 1287, wl.WALLS_Y, "fp32"), (701, 1333, wl.WALLS_Y, "fp16"),
    (1040, 581, wl.PERIODIC, "fp16"), (1741, 1757, wl.WALLS_Y, "fp16")])
def test_large_tiled_lattices_match_oracle(nx, ny, bc, precision):
    from paper_1507_03521_amd import Lattice
    from windows import compare_windows
    print(f"case large tiles {nx}x{ny} bc={bc} {precision}", flush=True)
    pb = wl.droplet64().with_(nx=nx, ny=ny, bc=bc, gx=2e-5, gy=-1e-5, rho_ref=0.3)
    f, g = wl.random_state(nx, ny, seed=nx * 7 + ny)
    lat = Lattice(pb.as_dict(), np.full((ny, nx), 0.5), precision=precision, device="cuda:0")
    assert 2 * lat.state_bytes <= (220 if precision == "fp64" else 224) << 20
    lat.set_state(f, g)
    before = tuple(t.cpu() for t in lat.get_state())
    fixed = precision != "fp64"
    total = q229_total(lat.save_raw(), precision, nx, ny) if fixed else 0
    lat.step(2)
    # corners, edges and the interior; columns wrap, rows of a periodic
    # lattice are compared away from its first and last ones
    ys = (0, ny // 2 - 3, ny - 12) if bc == wl.WALLS_Y else (11, ny // 2 - 3, ny - 23)
    compare_windows(pb, before, lat.get_state(), [(y, x) for y in ys for x in (0, nx // 3, nx - 7)],
                    2, TOL[precision])
    if fixed:
        assert q229_total(lat.save_raw(), precision, nx, ny) == total
