"""Waves of fewer than 64 rays (spread_rays in cast.hip): the rays of a cast,
and every derived product, do not depend on how many of them share a wave.
The first n pixels of a sky cast alone (1 to 64 rays a wave, ragged ends)
against the same rays within one cast of 140,000 (64 a wave), bit for bit."""
import pytest

import synth

pytestmark = pytest.mark.gpu
COSMO = (0.3, 0.7, 0.7)
SIZES = [1, 3, 1023, 1025, 2049, 5003, 65537]


@pytest.mark.parametrize("name,adaptive,spc", [("gauss32", False, 3), ("amr_halo_small", True, 2)])
def test_rays_do_not_depend_on_their_wave(name, adaptive, spc):
    import torch

    import paper_2111_08744_amd as M
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    cells = synth.make_cells(name)
    grid = M.Grid(cells, COSMO)
    obs = [0.47 * cells.box] * 3

    def cfg(n, **kw):
        return M.CastConfig(obs, 0.02, 128, pix_first=[17], pix_count=[n], steps_per_cell=spc, adaptive=adaptive,
                            schedule=1, **kw)

    def beam(n):
        return M.infinitesimal_beam(grid, cfg(n))

    runs = {"cic": lambda n: M.cast(grid, cfg(n)), "tsc": lambda n: M.cast(grid, cfg(n, order=2)),
            "ngp": lambda n: M.cast(grid, cfg(n, order=0)), "iso_chi": lambda n: M.cast(grid, cfg(n, stop_surface="chi")),
            "ckpt": lambda n: M.cast(grid, cfg(n, checkpoint_every=8)), "diff": lambda n: M.cast(grid, cfg(n, dphidl="diff")),
            "jacobian": lambda n: M.jacobian(grid, cfg(n)), "beam": beam, "born": lambda n: M.born_beam(grid, cfg(n))}
    for tag, run in runs.items():
        print(name, tag, flush=True)
        whole = run(140000)
        for n in SIZES:
            part = run(n)
            for k, v in part.items():
                if not k.startswith("_"):
                    w = whole[k][:n]
                    assert torch.equal(v.nan_to_num(), w.nan_to_num()) and torch.equal(v.isnan(), w.isnan()), (tag, n, k)
