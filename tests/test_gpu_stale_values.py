"""mpath_adjoint after the cell values changed in the cells around the observer
alone: the path's last segment, replayed from its stored checkpoint, is as
before, the path itself is not.  A Jacobian asked for alone or together with
the cell gradient is refused alike: ray_status 2 and NaN."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
COSMO = (0.3, 0.7, 0.7)


# 48 rays take four lanes each, 20,000 one
@pytest.mark.parametrize("nside,count", [(2, 48), (64, 20000)])
@pytest.mark.parametrize("cells", [False, True])
def test_values_changed_near_the_observer(nside, count, cells):
    import torch

    import paper_2111_08744_amd as M
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    tree = synth.make_cells("gauss32")
    grid = M.Grid(tree, COSMO)
    obs = np.full(3, 0.47 * tree.box)
    cfg = M.CastConfig(obs, 0.4 * tree.box, nside, stop_kind="chi", pix_first=[0], pix_count=[count], steps_per_cell=4,
                       checkpoint_every=8)
    out = M.cast(grid, cfg)
    ones = {"dL_dalpha": torch.ones(count, 2, device="cuda"), "dL_dz": torch.ones(count, device="cuda", dtype=torch.float64)}
    kw = {"jacobian": True, "cells": cells, **(ones if cells else {})}
    print(nside, count, cells, flush=True)
    res = M.adjoint(grid, cfg, out, **kw)
    assert int((res["ray_status"] != 0).sum()) == 0 and bool(torch.isfinite(res["jac"]).all())
    values = np.concatenate([tree.phi[:, None], tree.grad], 1).astype(np.float32)
    x = (tree.ijk + 0.5) * (tree.box / tree.n0)
    near = np.abs(x - obs).max(1) < 0.1 * tree.box
    values[near] *= 1.5
    grid.set_values(torch.from_numpy(values).cuda())
    res = M.adjoint(grid, cfg, out, **kw)
    assert bool((res["ray_status"] == 2).all())
    assert bool(torch.isnan(res["jac"]).all()) and bool(torch.isnan(res["dz_dtheta"]).all())
