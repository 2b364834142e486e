"""The per-ray derivatives of mpath_adjoint, mpath_cast_jacobian and the finder over a long path:
3,000 steps to z = 1 on a uniform grid, against the oracle's complex step.
Stage quantities are float32 on both the tangents' and the reverse sweep's
way, one rounding (6e-8 relative) each; what a step adds is summed in double
precision, so the error stays at a rounding or two of the sum however many
steps there are.  Bar: 1.8e-7 (three half-ulps) of the rms of dz5/dtheta on
the median.  (Summed in float32 the 3,000 roundings walk to four times the
error.)"""
import numpy as np
import pytest

import oracle as O
import synth
from parity import oracle_dirs

pytestmark = pytest.mark.gpu
COSMO = (0.3, 0.7, 0.7)


@pytest.fixture(scope="module")
def case():
    import torch

    import paper_2111_08744_amd as M
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    cells = synth.make_cells("gauss64")
    return M, cells, M.Grid(cells, COSMO), [0.5 * cells.box] * 3


@pytest.mark.parametrize("call", ["adjoint", "jacobian"])
def test_redshift_derivative_of_a_long_path(case, call):
    M, cells, grid, obs = case
    if call == "adjoint":
        cfg = M.CastConfig(obs, 1.0, 4, [0], [96], steps_per_cell=10, checkpoint_every=32)
        out = M.cast(grid, cfg)
        res = M.adjoint(grid, cfg, out, jacobian=True)
    else:
        out = res = M.jacobian(grid, M.CastConfig(obs, 1.0, 4, [0], [96], steps_per_cell=10))
    dz = res["dz_dtheta"].cpu().numpy().astype(np.float64)
    assert (out["n_steps"].cpu().numpy() > 2500).all()
    p = O.params(obs, z_src=1.0, steps_per_cell=10, adaptive=False)
    field, c = O.Field.grid(cells), O.cosmo(*COSMO)
    _, ref, rec = O.jacobian_cs(lambda d, t: O.cast_cs(field, c, p, d, dtheta=t), oracle_dirs(4, [0], [96]))
    err, size = np.median(np.abs(dz - ref)), np.sqrt(np.mean(ref ** 2))
    print(err, size, err / size, flush=True)
    assert err <= 1.8e-7 * size


def test_finder_takes_the_same_derivatives(case):
    """The finder's matrices are those of mpath_adjoint along its directions,
    with sources at one distance: to a rounding of float32 of the entry and of
    the lensing terms' rms (the distances, and with them the ends, agree to
    rounding in double precision)."""
    import torch
    M, cells, grid, obs = case
    n, chi = 300, 4.0 * cells.box
    v = np.random.default_rng(2).standard_normal((n, 3))
    src = np.asarray(obs) + v / np.linalg.norm(v, axis=1, keepdims=True) * chi
    res = M.find_geodesics(grid, obs, src, steps_per_cell=10, tol=1e-9)
    assert int((res["status"] != 0).sum()) == 0
    cfg = M.CastConfig(obs, chi, 1, pix_count=[n], dirs=res["theta"].contiguous(), stop_kind="chi", steps_per_cell=10,
                       checkpoint_every=32)
    adj = M.adjoint(grid, cfg, M.cast(grid, cfg), jacobian=True)
    for a, b, unlensed in ((res["dz_dtheta"], adj["dz_dtheta"], 0.0),
                           (res["A"], adj["jac"], torch.eye(2, device="cuda", dtype=torch.float64))):
        b = b.double()
        d = (a.double() - b).abs()
        print(float(d.max()), float(d.median()), flush=True)
        assert bool((d <= 1.2e-7 * (b.abs() + (b - unlensed).square().mean().sqrt())).all())
