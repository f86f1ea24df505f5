"""Checkpoint segments that read and write raw snapshots in place of the
context's state (lbm_segment), bitwise against the calls with copies, on each
path that a step can take; and what lbm_init leaves beyond the planes."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


def _lat(nx, ny, precision, flags=0, seed=1):
    from paper_1507_03521_amd import Lattice
    pb = wl.droplet64().with_(nx=nx, ny=ny, bc=wl.WALLS_Y, gy=-1e-5, rho_ref=0.3)
    lat = Lattice(pb.as_dict(), np.full((ny, nx), 0.5), precision=precision, flags=flags,
                  device="cuda:0")
    f, g = wl.random_state(nx, ny, seed=seed)
    lat.set_state(f, g)
    return lat


# two-step tiles, one-step tiles, row sweeps (two steps and, odd, one), unfused
@pytest.mark.parametrize("n", [1, 2, 5])
@pytest.mark.parametrize("nx,ny,precision,flags", [
    (40, 37, "fp64", 0), (300, 290, "fp32", 0), (40, 37, "fp16", 0), (1000, 900, "fp64", 0),
    (1203, 1300, "fp32", 0), (60, 50, "fp32", 2)])
def test_segment_matches_copies(nx, ny, precision, flags, n):
    from paper_1507_03521_amd import QilbmError
    print(f"case segment {nx}x{ny} {precision} flags={flags} n={n}", flush=True)
    a, b = _lat(nx, ny, precision, flags), _lat(nx, ny, precision, flags)
    nb = a.record_bytes
    ra, rb = ([torch.zeros(nb, dtype=torch.uint8, device="cuda") for _ in range(n)]
              for _ in range(2))
    s0 = a.save_raw()
    a.step_records(ra)
    s1 = a.save_raw()
    a.step(n)
    # b: the state's own, then into a snapshot, then from it
    t1 = torch.zeros_like(s1)
    b.segment(n, records=b.record_array(rb), dst=t1)
    for call in (lambda: b.step(1), lambda: b.moments(("phi",)), b.mass, b.get_state, b.save_raw,
                 lambda: b.segment(1)):
        with pytest.raises(QilbmError) as e:
            call()
        assert e.value.status == -5
    # snapshots start zeroed here, padding included, as the states do
    assert torch.equal(s1, t1)
    assert all(torch.equal(x, y) for x, y in zip(ra, rb))
    b.segment(n, src=t1, t=n)
    assert b.time == a.time == 2 * n
    assert torch.equal(a.save_raw(), b.save_raw())
    # and again from the first snapshot, with the records
    for r in rb:
        r.zero_()
    b.segment(n, src=s0, t=0, records=b.record_array(rb))
    assert b.time == n and torch.equal(b.save_raw(), s1)
    assert all(torch.equal(x, y) for x, y in zip(ra, rb))


def test_segment_refuses_bad_arguments():
    lat = _lat(40, 37, "fp64")
    raw = torch.zeros(lat.state_bytes + 256, dtype=torch.uint8, device="cuda")
    seg = lat.lib.lbm_segment
    p = raw.data_ptr()
    none = ctypes.POINTER(ctypes.c_void_p)()
    assert seg(lat.ctx, None, 0, 0, none, None) == -1
    assert seg(lat.ctx, p, -1, 1, none, None) == -1
    assert seg(lat.ctx, p + 8, 0, 1, none, None) == -1
    assert seg(lat.ctx, None, 0, 1, none, p + 8) == -1
    assert seg(lat.ctx, p, 0, 1, none, p) == -1
    assert lat.time == 0


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16"])
def test_raw_padding_is_zero_on_a_used_workspace(precision):
    """Equal states give equal snapshots whatever the workspace held (odd node
    counts: the planes end inside a word of the binary16 planes)."""
    raws = []
    for fill in (0xAB, 0x55):
        lat = _lat(41, 37, precision)
        dirty = torch.full_like(lat.workspace, fill)
        lat.workspace.copy_(dirty)
        from paper_1507_03521_amd import _lib
        ctx = ctypes.c_void_p()
        _lib.check(lat.lib.lbm_init(ctypes.byref(ctx), ctypes.byref(lat.params),
                                    lat.workspace.data_ptr(), lat.workspace.numel(),
                                    lat.phi0.data_ptr(),
                                    ctypes.c_void_p(lat.stream.cuda_stream)), "lbm_init")
        lat.lib.lbm_destroy(lat._ctx)
        lat._ctx = ctx
        got = [lat.save_raw()]
        for k in (1, 1, 2):
            lat.step(k)
            got.append(lat.save_raw())
        raws.append(got)
    assert all(torch.equal(x, y) for x, y in zip(*raws))
