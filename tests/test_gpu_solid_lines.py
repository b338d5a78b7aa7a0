"""Solid nodes over several steps of one call: the later steps leave cache
lines of solid nodes alone (the second buffer holds them since the first
step).  lbm_step(h, 5) equals five lbm_step(h, 1) bit for bit, the solid
nodes included, with solid runs shorter and longer than a line, rows that
are not whole lines, both layouts, and the state replaced between calls."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0811_4593_amd import lbm, workloads  # noqa: E402

STORAGES = [lbm.LBM_STORE_F64, lbm.LBM_STORE_F32, lbm.LBM_STORE_F16_DEV, lbm.LBM_STORE_F16_DEV_SR]


def _solid(nx, ny, nz):
    s = np.zeros((nz, ny, nx), np.uint8)
    s[:, 1] = 1                      # whole rows
    s[:, 3, 5:9] = 1                 # less than a line
    s[1, 4, nx // 2:] = 1            # a run that starts inside a line
    s[2] = 1                         # a whole plane
    return s


def _states(nx, ny, nz):
    w = np.array([1 / 18] * 6 + [1 / 36] * 12 + [1 / 3])[:, None, None, None]
    return [w * workloads.perturbation((19, nz, ny, nx), seed, 0.05) for seed in (1, 2)]


@pytest.mark.parametrize("geometry", [False, True], ids=["mask", "geometry"])
@pytest.mark.parametrize("layout", [0, 1], ids=["population-major", "row-major"])
@pytest.mark.parametrize("nx", [64, 150])
@pytest.mark.parametrize("storage", STORAGES, ids=lambda s: lbm.STORAGE_NAMES[s])
def test_steps_in_one_call_equal_single_calls(storage, nx, layout, geometry):
    ny, nz = 6, 5
    solid = _solid(nx, ny, nz)
    got = []
    for calls in ((5, 4), (1,) * 9):
        h = lbm.lbm_create(nx, ny, nz, 0.9, 1.0, None, storage, torch.cuda.current_stream())
        try:
            lbm.lbm_set_layout(h, layout)
            if geometry:
                lbm.lbm_set_geometry(h, workloads.cells_from_solid(solid))
            else:
                lbm.lbm_set_solid_mask(h, solid)
            out = np.empty((19, nz, ny, nx))
            done = 0
            states = _states(nx, ny, nz)
            lbm.lbm_set_populations(h, states[0])
            for n in calls:
                lbm.lbm_step(h, n)
                done += n
                if done == 5:
                    first = lbm.lbm_get_populations(h, out).copy()
                    lbm.lbm_set_populations(h, states[1])
            got.append((first, lbm.lbm_get_populations(h, out).copy()))
        finally:
            lbm.lbm_destroy(h)
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
