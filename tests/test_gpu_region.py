"""Rays that run along the faces of the cached stencil regions (FieldCache in
device.h): the dual cells' faces are the planes through cell centres, so an
observer at a cell centre puts every in-plane ray exactly on them, and the
reverse sweep, whose replay reaches the same points with another cache
history, must retrace them bit for bit.  Oracle and bars of parity.py."""
import numpy as np
import pytest

import oracle as O
import synth
from parity import compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu
COSMO = (0.3, 0.7, 0.7)


@pytest.mark.parametrize("name,adaptive,spc", [("gauss32", False, 4), ("amr_halo_small", True, 4)])
@pytest.mark.parametrize("offset", [0.5, 0.25, 0.0])
def test_rays_in_the_planes_of_region_faces(name, adaptive, spc, offset):
    import torch

    import paper_2111_08744_amd as M
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    cells = synth.make_cells(name)
    grid = M.Grid(cells, COSMO)
    # on the coarse cell centre, on a level-1 centre, on a cell face
    obs = [(cells.n0 // 2 + offset) * cells.box / cells.n0] * 3
    print(name, offset, flush=True)
    cfg = M.CastConfig(obs, 0.2, 4, steps_per_cell=spc, adaptive=adaptive)
    o = run_oracle(O.Field.grid(cells), O.cosmo(*COSMO), obs, 0.2, 4, [0], [192], spc, adaptive)
    compare(run_gpu(grid, cfg), o)
    cfgk = M.CastConfig(obs, 0.2, 4, steps_per_cell=spc, adaptive=adaptive, checkpoint_every=16)
    res = M.adjoint(grid, cfgk, M.cast(grid, cfgk), jacobian=True)
    assert int((res["ray_status"] != 0).sum()) == 0
    assert np.isfinite(res["jac"].cpu().numpy()).all()
