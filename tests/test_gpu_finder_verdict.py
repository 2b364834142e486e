"""Whether a source has converged is decided once an iteration: with the
tolerance on a source's own separation, or next to it, every source either
stays where it is and reports that iteration, or takes a Newton step by its
own matrix.  The workspace holds NaN, so that a source that moves by a matrix
nobody wrote ends as NaN.  And the matrix step of more sources on a tree than
take four lanes each."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
COSMO = (0.3, 0.7, 0.7)


def _find(M, grid, obs, src, **kw):
    """find_geodesics with a workspace of NaN; arrays on the host."""
    import torch
    ws = M.find_geodesics(grid, obs, src, steps_per_cell=3, max_iter=1, adaptive=kw.get("adaptive", False))["_ws"]
    ws.fill_(255)
    torch.cuda.synchronize()
    res = M.find_geodesics(grid, obs, src, steps_per_cell=3, ws=ws, **kw)
    assert res["_ws"] is ws
    return {k: v.cpu().numpy() for k, v in res.items() if not k.startswith("_")}


@pytest.mark.parametrize("levels", [0, 3])
def test_one_verdict_an_iteration(levels):
    import torch

    import paper_2111_08744_amd as M
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    cells = synth.random_amr_cells(16, 125.0, levels, seed=5) if levels else synth.make_cells("gauss32")
    grid = M.Grid(cells, COSMO)
    n = 500
    v = np.random.default_rng(4).standard_normal((n, 3))
    obs = np.full(3, 0.47 * cells.box)
    src = obs + v / np.linalg.norm(v, axis=1, keepdims=True) * 0.2 * cells.box
    start = _find(M, grid, obs, src, max_iter=1, identity_iters=0, tol=1.0)       # all converge where they start
    assert (start["n_iter"] == 0).all()
    sep = start["sep"]
    order = np.argsort(sep)
    for k in order[[0, 1, n // 4, n // 2, n - 2, n - 1]]:
        for tol in (np.nextafter(sep[k], 0.0), sep[k], np.nextafter(sep[k], 1.0)):
            print(levels, k, tol, flush=True)
            res = _find(M, grid, obs, src, max_iter=1, identity_iters=0, tol=tol)
            stay = (res["theta"] == start["theta"]).all(1)
            assert np.array_equal(stay, res["n_iter"] == 0)
            # apart from the source on the line itself the verdict is known
            sure = np.arange(n) != k
            assert np.array_equal(stay[sure], sep[sure] < tol)
            # A is within a per cent of the identity at this distance: a step is
            # the separation to a few per cent
            step = np.linalg.norm(res["theta"] - start["theta"], axis=1)[~stay]
            assert (np.abs(step / sep[~stay] - 1.0) < 0.05).all()


def test_matrix_step_of_one_lane_a_ray_on_a_tree():
    """Rays past the line of four lanes each (one a lane, adjoint_kernel on a
    tree) against the same sources in parts that take four.  The matrices are
    single-precision on both sides (1e-6 relative each), and the first step is
    the longest, so the roots agree to 2e-6 of it, and the rounding of
    double-precision directions."""
    import torch

    import paper_2111_08744_amd as M
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    cells = synth.random_amr_cells(16, 125.0, 3, seed=5)
    grid = M.Grid(cells, COSMO)
    n = 64 * torch.cuda.get_device_properties(0).multi_processor_count + 3
    v = np.random.default_rng(9).standard_normal((n, 3))
    obs = np.full(3, 0.47 * cells.box)
    src = obs + v / np.linalg.norm(v, axis=1, keepdims=True) * 0.2 * cells.box

    def find(s, tol=1e-9):
        print(len(s), flush=True)
        return _find(M, grid, obs, s, adaptive=True, identity_iters=0, tol=tol)

    whole, parts = find(src), [find(src[:n // 2]), find(src[n // 2:])]
    both = {k: np.concatenate([p[k] for p in parts]) for k in whole}
    assert np.array_equal(whole["status"], both["status"]) and np.array_equal(whole["n_iter"], both["n_iter"])
    first = find(src, 1.0)["sep"].max()
    assert np.abs(whole["theta"] - both["theta"]).max() <= 2e-6 * first + 1e-15
