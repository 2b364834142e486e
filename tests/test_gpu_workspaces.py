"""Sizes of the reverse mode's workspaces: the segment's states and the cell
cotangents, with the Jacobian's tangents in the states' place, and results
that do not depend on how far the two overlap."""
import ctypes as C

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
COSMO = (0.3, 0.7, 0.7)


@pytest.fixture(scope="module")
def case():
    import torch

    import paper_2111_08744_amd as M
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    cells = synth.make_cells("gauss32")
    return M, cells, M.Grid(cells, COSMO)


def _cfg(M, cells, n, K):
    return M.CastConfig([0.47 * cells.box] * 3, 0.2 * cells.box, 64, stop_kind="chi", pix_first=[0], pix_count=[n],
                        steps_per_cell=3, checkpoint_every=K)


def _bytes(fn, *args):
    from paper_2111_08744_amd import _abi
    out = C.c_size_t()
    _abi.check(getattr(_abi.lib(), fn)(*args, C.byref(out)), fn)
    return out.value


def test_adjoint_workspace_is_the_states_and_the_cells(case):
    M, cells, grid = case
    for n in (1, 1000, 30001):
        for K in (1, 2, 4, 32):
            got = _bytes("mpath_adjoint_workspace_bytes", grid.handle, C.byref(_cfg(M, cells, n, K).desc()))
            assert got <= (40 * K if K >= 4 else 144) * n + 16 * cells.n_cells + 2 * 256, (n, K, got)


def test_finder_workspace_is_the_cast_the_sweep_and_tables(case):
    from paper_2111_08744_amd import _abi
    M, cells, grid = case
    n, K = 5000, 16
    chi = 0.2 * cells.box
    v = np.random.default_rng(1).standard_normal((n, 3))
    obs = np.full(3, 0.47 * cells.box)
    src = obs + v / np.linalg.norm(v, axis=1, keepdims=True) * chi
    f = _abi.mpath_finder_desc()
    f.obs_pos, f.n_src, f.src_pos, f.order, f.steps_per_cell = obs.ctypes.data, n, src.ctypes.data, 1, 3
    f.max_steps, f.tol, f.max_iter, f.identity_iters, f.checkpoint_every = 1 << 40, 1e-9, 5, 0, K
    d = _cfg(M, cells, n, K).desc()
    parts = sum(_bytes(k, grid.handle, C.byref(d)) for k in ("mpath_cast_workspace_bytes", "mpath_adjoint_workspace_bytes"))
    got = _bytes("mpath_find_geodesics_workspace_bytes", grid.handle, C.byref(f))
    assert got <= parts + 80 * n + 12 * 256, (got, parts)


@pytest.mark.parametrize("n", [1, 47, 17000])
def test_results_do_not_depend_on_the_overlap(case, n):
    """The matrices bit for bit, the cells to their atomics' order (sums of up
    to 1e4 float32 terms a cell, 1e2 roundings of the norm)."""
    import torch
    M, cells, grid = case
    gen = torch.Generator("cuda").manual_seed(1)
    ga = torch.randn(n, 2, device="cuda", generator=gen)
    gz = torch.randn(n, device="cuda", generator=gen, dtype=torch.float64)
    ref = None
    for K in (64, 4, 3, 1):
        print(n, K, flush=True)
        cfg = _cfg(M, cells, n, K)
        out = M.cast(grid, cfg)
        both = M.adjoint(grid, cfg, out, dL_dalpha=ga, dL_dz=gz, jacobian=True, cells=True)
        cells_alone = M.adjoint(grid, cfg, out, dL_dalpha=ga, dL_dz=gz, cells=True)["dL_dvalues"].double()
        alone = M.adjoint(grid, cfg, out, jacobian=True)
        assert int((both["ray_status"] != 0).sum()) == 0
        ref = ref or (both["jac"], both["dz_dtheta"], both["dL_dvalues"].double())
        for r in (both, alone):
            assert torch.equal(r["jac"], ref[0]) and torch.equal(r["dz_dtheta"], ref[1])
        for g in (both["dL_dvalues"].double(), cells_alone):
            assert float((g - ref[2]).norm()) <= 6e-6 * float(ref[2].norm())
