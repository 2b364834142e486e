"""Casts whose rays take four lanes each (by_quads in device.h) against the
persistent schedule, one lane per ray, bit for bit: rays that leave the box of
a non-periodic grid through every face and edge, partly filled waves, and the
numbers of rays on both sides of the rule's line."""
import dataclasses

import pytest

import synth

pytestmark = pytest.mark.gpu
COSMO = (0.3, 0.7, 0.7)


def _equal(M, grid, n, tag, **kw):
    import torch
    one, four = (M.cast(grid, M.CastConfig(nside=128, pix_first=[0], pix_count=[n], schedule=s, **kw)) for s in (2, 1))
    with_tangents = M.jacobian(grid, M.CastConfig(nside=128, pix_first=[0], pix_count=[n], **kw))
    for k, v in one.items():
        if not k.startswith("_"):
            assert torch.equal(v.view(torch.uint8), four[k].view(torch.uint8)), (tag, n, k)
            assert torch.equal(v.view(torch.uint8), with_tangents[k].view(torch.uint8)), (tag, n, k)
    return four


@pytest.mark.parametrize("levels", [0, 3])
@pytest.mark.parametrize("periodic", [True, False])
def test_four_lanes_a_ray(levels, periodic):
    import torch

    import paper_2111_08744_amd as M
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    if levels:
        cells = synth.random_amr_cells(16, 125.0, levels, seed=5, periodic=periodic)
    else:
        cells = dataclasses.replace(synth.make_cells("gauss32"), periodic=periodic)
    grid = M.Grid(cells, COSMO)
    for f in (0.47, 0.03):
        kw = dict(obs=[f * cells.box, 0.5 * cells.box, 0.6 * cells.box], stop=0.7 * cells.box, stop_kind="chi", steps_per_cell=3,
                  adaptive=levels > 0)
        for n in (1, 15, 17, 1025, 16391):
            print(levels, periodic, f, n, flush=True)
            out = _equal(M, grid, n, (levels, periodic, f), **kw)
        assert periodic or int((out["status"] != 0).sum()) > 0
    line = 64 * torch.cuda.get_device_properties(0).multi_processor_count * (4 if levels else 2)
    for n in (line, line + 1):
        _equal(M, grid, n, "line", **{**kw, "stop": 0.05 * cells.box})


@pytest.mark.parametrize("levels", [0, 3])
def test_cell_gradient_of_four_lanes_a_ray(levels):
    """The cell gradient is a sum over rays: of more rays than take four lanes
    each, and of their parts, which do.  Single-precision sums of up to 1e4
    terms a cell in another order: 1e2 roundings of 6e-8 of the norm."""
    import torch

    import paper_2111_08744_amd as M
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    cells = synth.random_amr_cells(16, 125.0, levels, seed=5) if levels else synth.make_cells("gauss32")
    grid = M.Grid(cells, COSMO)
    n = 64 * torch.cuda.get_device_properties(0).multi_processor_count
    gen = torch.Generator("cuda").manual_seed(3)
    ga = torch.randn(n + 3, 2, device="cuda", generator=gen)
    gz = torch.randn(n + 3, device="cuda", generator=gen, dtype=torch.float64)

    def gradient(lo, hi):
        cfg = M.CastConfig([0.47 * cells.box, 0.5 * cells.box, 0.6 * cells.box], 0.3 * cells.box, 128, stop_kind="chi",
                           pix_first=[lo], pix_count=[hi - lo], steps_per_cell=3, adaptive=levels > 0,
                           checkpoint_every=8)
        print(levels, lo, hi, flush=True)
        res = M.adjoint(grid, cfg, M.cast(grid, cfg), dL_dalpha=ga[lo:hi].contiguous(), dL_dz=gz[lo:hi].contiguous(),
                        jacobian=False, cells=True)
        assert int((res["ray_status"] != 0).sum()) == 0
        return res["dL_dvalues"].double()

    whole = gradient(0, n + 3)
    parts = gradient(0, 1) + gradient(1, 1030) + gradient(1030, n + 3)
    assert float((whole - parts).norm()) <= 6e-6 * float(whole.norm())


def test_finder_steps_of_four_lanes_a_ray():
    """The finder's Newton steps: the distortion matrices of more rays than
    take four lanes each against the same sources in two calls, whose rays do.
    The matrices are single-precision on both sides (1e-6 relative), and the
    last step is below 1e-7 rad of the root (tol), so the roots agree to 1e-13
    rad plus the rounding of double-precision directions."""
    import numpy as np
    import torch

    import paper_2111_08744_amd as M
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    cells = synth.make_cells("gauss32")
    grid = M.Grid(cells, COSMO)
    n = 64 * torch.cuda.get_device_properties(0).multi_processor_count + 3
    v = np.random.default_rng(9).standard_normal((n, 3))
    obs = np.full(3, 0.5 * cells.box)
    src = obs + v / np.linalg.norm(v, axis=1, keepdims=True) * 0.2 * cells.box

    def find(s):
        print(len(s), flush=True)
        res = M.find_geodesics(grid, obs, s, steps_per_cell=3, identity_iters=0, tol=1e-9)
        return {k: res[k].cpu() for k in ("theta", "n_iter", "status")}

    whole, parts = find(src), [find(src[:n // 2]), find(src[n // 2:])]
    both = {k: torch.cat([p[k] for p in parts]) for k in whole}
    assert torch.equal(whole["status"], both["status"]) and torch.equal(whole["n_iter"], both["n_iter"])
    assert float((whole["theta"] - both["theta"]).abs().max()) <= 1e-12


def test_automatic_schedule_of_many_observers():
    """On both sides of the number of rays where the automatic choice changes."""
    import torch

    import paper_2111_08744_amd as M
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    cells = synth.make_cells("gauss32")
    grid = M.Grid(cells, COSMO)
    line = 64 * 4 * 4 * torch.cuda.get_device_properties(0).multi_processor_count
    obs = [[f * cells.box] * 3 for f in (0.3, 0.6)]
    for n in (line, line + 1):
        print(n, flush=True)
        auto, static = (M.cast(grid, M.CastConfig(obs, [0.03 * cells.box, 0.06 * cells.box], 256, stop_kind="chi",
                                                  pix_first=[0, 5], pix_count=[1000, n - 1000], steps_per_cell=3,
                                                  schedule=s)) for s in (0, 1))
        for k, v in auto.items():
            if not k.startswith("_"):
                assert torch.equal(v.view(torch.uint8), static[k].view(torch.uint8)), (n, k)
