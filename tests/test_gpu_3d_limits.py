"""Three-dimensional lattices at the ends of what the context accepts."""
import numpy as np
import pytest
import torch

import workloads as wl
from test_gpu_3d import _problem

pytestmark = pytest.mark.gpu


def test_lattice_whose_tiles_exceed_one_grid_dimension():
    """3 x 5 x (2^25 + 64) nodes (the limit is 2^29 in all): tiles 16 nodes
    wide and 4 deep have 2^32 lanes and more, beyond one dimension of a launch.
    The initial phi repeats every 64 layers, and so do its steps: every period
    equals the same steps of a lattice of 64 layers, to rounding (binary32 phi
    of order one and a few steps: 1e-6)."""
    from paper_1507_03521_amd import Lattice3D
    nz, period = 2 ** 25 + 64, 64
    dev = torch.device("cuda:0")
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 215e9:
        pytest.skip("needs 215 GB of free device memory")
    rng = np.random.default_rng(8)
    one = torch.tensor(0.2 + 0.6 * rng.random((period, 5, 3)), device=dev)
    out = []
    for n in (period, nz):
        pb = _problem(3, 5, n, wl.PERIODIC, (1e-6, -2e-6, -1e-5))
        phi0 = one if n == period else one.repeat(n // period, 1, 1)
        lat = Lattice3D(pb.as_dict(), phi0, precision="fp32", device=dev)
        lat.phi0 = None
        del phi0
        lat.step(2)
        out.append(lat.moments(("phi",))["phi"])
        lat.close()
        del lat
        torch.cuda.empty_cache()
    small, large = out
    assert float((small - one).abs().max()) > 1e-3         # the steps move it
    worst = max(float((part.view(-1, period, 5, 3) - small).abs().max())
                for part in large.split(period * 2 ** 15))
    print(f"  worst difference to the 64-layer lattice {worst:.2e}", flush=True)
    assert worst <= 1e-6
    del out, small, large
    torch.cuda.empty_cache()
