"""The autotuner times the launch that will run: its sample of a cast whose
rays take one lane each takes one lane a ray too, though the sample's own
number of rays would take four (and the reverse for a cast that takes four)."""
import pytest

import synth

pytestmark = pytest.mark.gpu
COSMO = (0.3, 0.7, 0.7)


def _kernels(run):
    """Names of the GPU kernels that run() launches."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        run()
        torch.cuda.synchronize()
    return {e.name for e in prof.events()}


@pytest.mark.parametrize("levels", [0, 3])
def test_sample_takes_the_form_of_the_launch(levels):
    import torch

    import paper_2111_08744_amd as M
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    cells = synth.random_amr_cells(16, 125.0, levels, seed=5) if levels else synth.make_cells("gauss32")
    grid = M.Grid(cells, COSMO)
    most = 64 * torch.cuda.get_device_properties(0).multi_processor_count * (4 if levels else 2)   # four lanes a ray
    for n in (most, most + 8):
        cfg = M.CastConfig([0.5 * cells.box] * 3, 0.03 * cells.box, 256, stop_kind="chi", pix_first=[0], pix_count=[n],
                           steps_per_cell=3, adaptive=levels > 0)
        print(levels, n, flush=True)
        static = _kernels(lambda: M.cast(grid, M.CastConfig([0.5 * cells.box] * 3, 0.03 * cells.box, 256, stop_kind="chi",
                                                            pix_first=[0], pix_count=[n], steps_per_cell=3,
                                                            adaptive=levels > 0, schedule=1)))
        cast = {k for k in static if "cast_quad_kernel" in k or "cast_static_kernel" in k}
        assert len(cast) == 1 and ("cast_quad_kernel" in list(cast)[0]) == (n == most)
        tuned = _kernels(lambda: M.autotune(grid, cfg, sample_div=8))
        assert {k for k in tuned if "cast_quad_kernel" in k or "cast_static_kernel" in k} == cast
        assert any("cast_persistent_kernel" in k for k in tuned)
