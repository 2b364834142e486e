"""The Hessian of the infinitesimal and Born beams on uniform grids: the mixed
entry of the distortion matrices, whose float32 value is rounded at 6e-8 of
itself and not of one, and the edges of a non-periodic box."""
import dataclasses

import numpy as np
import pytest

import oracle as O
import synth

pytestmark = pytest.mark.gpu
COSMO = (0.3, 0.7, 0.7)


def _cells(name, **kw):
    """Cell values as the grid holds them."""
    c = synth.make_cells(name)
    return dataclasses.replace(c, phi=c.phi.astype(np.float32).astype(np.float64),
                               grad=c.grad.astype(np.float32).astype(np.float64), **kw)


@pytest.mark.parametrize("kind", ["infinitesimal", "born"])
def test_mixed_entry(kind):
    """Rms error of A12 over 768 rays against the oracle (FP64 throughout), as
    a part of its rms: 2e-8 for its own rounding to float32 (uniform, half an
    ulp at most 6e-8), and for a sample's H, interpolated in float32 from
    differences of float32 cells, up to six roundings of 3e-8 / sqrt(3) whose
    mean over a ray's samples is smaller: together below 5e-8."""
    import torch

    import paper_2111_08744_amd as M
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    cells = _cells("gauss64")
    obs, z, nside = [0.5 * cells.box] * 3, 0.1, 8
    grid = M.Grid(cells, COSMO)
    cfg = M.CastConfig(obs, z, nside, steps_per_cell=10)
    A = getattr(M, kind + "_beam")(grid, cfg)["A"].cpu().numpy().astype(np.float64)
    p = O.params(obs, z_src=z, steps_per_cell=10, adaptive=False)
    ref, _ = getattr(O, kind)(O.Field.grid(cells), O.cosmo(*COSMO), p, O.pix2vec_nest(nside, np.arange(len(A))))
    err, size = (np.sqrt(np.mean(x ** 2)) for x in (A[:, 0, 1] - ref[:, 0, 1], ref[:, 0, 1]))
    print(kind, err, size, err / size, flush=True)
    assert err <= 5e-8 * size


@pytest.mark.parametrize("at", [(0.2, 16.3, 16.7), (16.1, 31.8, 16.7), (0.3, 31.9, 0.1), (1.2, 30.6, 15.5), (16, 16, 16)])
def test_edges_of_a_box(at):
    """Lines that start, run and end where a probe, or the point itself, has no
    complete stencil: such rows of H are zero."""
    import torch

    import paper_2111_08744_amd as M
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    cells = _cells("gauss32", periodic=False)
    obs = [c * cells.box / cells.n0 for c in at]
    grid = M.Grid(cells, COSMO)
    chi = 0.3 * cells.box
    print(at, flush=True)
    res = M.born_beam(grid, M.CastConfig(obs, chi, 4, stop_kind="chi", steps_per_cell=4))
    p = O.params(obs, chi=chi, steps_per_cell=4, adaptive=False)
    ref, rec = O.born(O.Field.grid(cells), O.cosmo(*COSMO), p, O.pix2vec_nest(4, np.arange(192)))
    A, status = res["A"].cpu().numpy(), res["status"].cpu().numpy()
    assert np.array_equal(status, rec["status"]) and (status == 0).any()
    ok = status == 0
    # float32 entries of order one, and float32 H on a signal of a per cent
    assert np.abs(A[ok] - ref[ok]).max() <= 1.2e-7 + 1e-6 * np.abs(ref[ok] - np.eye(2)).max()
    assert np.isnan(A[~ok]).all()
