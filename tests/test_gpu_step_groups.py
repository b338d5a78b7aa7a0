"""Several steps per launch without being asked for (lbm_step with one step
per pass, and chunks of a single batch job): blocks of steps on small
lattices and passes of two steps on larger ones give, bit for bit, the state
of single sweeps (lbm_step one step at a time), in the buffer that single
sweeps end in, on lattices around the block and tile edges, with every node
class, pressure faces, a body force and the rule without N."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0811_4593_amd import lbm, serving, workloads  # noqa: E402

STORAGES = [lbm.LBM_STORE_F64, lbm.LBM_STORE_F32, lbm.LBM_STORE_F16_DEV, lbm.LBM_STORE_F16_DEV_SR]
INT_OF = {8: torch.int64, 4: torch.int32, 2: torch.int16}
W = np.array([1 / 18] * 6 + [1 / 36] * 12 + [1 / 3])[:, None, None, None]

SMALL = [
    workloads.all_classes_lattices()[2],
    workloads.all_classes_lattices()[4],
    workloads.pressure_classes_lattices()[1],
    workloads.duct(17, 9, 13, (0.03, -0.02, 0.01), 0.8),   # blocks cut short on every axis
    workloads.couette(16, 16, 32),
    workloads.duct(65, 21, 30, (0.04, 0.01, 0.01), 0.7),   # bars cut short, above the cubes' range
    workloads.LatticeSpec(3, 3, 200, 0.9, {}, name="periodic_3x3x200"),
    workloads.LatticeSpec(2, 40, 7, 0.9, {}, name="periodic_2x40x7"),  # too thin for blocks
]


def _pair(spec, storage, layout, force=None, no_n=False):
    """Two equal lattices on caller-owned buffers, with those buffers."""
    esize = lbm.lbm_element_bytes(storage)
    n = max(lbm.lbm_buffer_elements(spec.nx, spec.ny, spec.nz, storage, k) for k in (0, 1))
    f0 = W * workloads.perturbation((19, spec.nz, spec.ny, spec.nx), 5, 0.05)
    out = []
    for _ in range(2):
        bufs = [torch.zeros(n, dtype=INT_OF[esize], device="cuda") for _ in range(2)]
        h = lbm.lbm_create_on_buffers(spec.nx, spec.ny, spec.nz, spec.tau, 1.0, None, storage,
                                      torch.cuda.current_stream(), bufs[0], bufs[1], n * esize)
        lbm.lbm_set_layout(h, layout)
        serving.apply_bc(h, spec)
        if force is not None:
            lbm.lbm_set_body_force(h, force)
        if no_n:
            lbm.lbm_set_rule_options(h, lbm.LBM_RULE_NO_TRANSVERSE)
        lbm.lbm_set_populations(h, f0)
        out.append((h, bufs))
    return out


def _compare(spec, storage, layout, counts, **more):
    (a, abufs), (b, bbufs) = _pair(spec, storage, layout, **more)
    try:
        for n in counts:
            lbm.lbm_step(a, n)
            for _ in range(n):
                lbm.lbm_step(b, 1)
            torch.cuda.synchronize()
            assert lbm.lbm_get_step(a) == lbm.lbm_get_step(b)
            which = [lbm.lbm_state_buffer(h) == bufs[0].data_ptr() for h, bufs in ((a, abufs), (b, bbufs))]
            assert which[0] == which[1]
            got = [np.empty((19, spec.nz, spec.ny, spec.nx)) for _ in range(2)]
            lbm.lbm_get_populations(a, got[0])
            lbm.lbm_get_populations(b, got[1])
            np.testing.assert_array_equal(got[0], got[1], err_msg=f"{spec.name} after {n} steps")
    finally:
        lbm.lbm_destroy(a)
        lbm.lbm_destroy(b)


@pytest.mark.parametrize("layout", [0, 1], ids=["population-major", "row-major"])
@pytest.mark.parametrize("storage", STORAGES, ids=lambda s: lbm.STORAGE_NAMES[s])
@pytest.mark.parametrize("spec", SMALL, ids=lambda s: s.name)
def test_small_lattices(spec, storage, layout):
    _compare(spec, storage, layout, (3, 2, 7, 10), force=(1e-5, -2e-5, 3e-5))


@pytest.mark.parametrize("storage", STORAGES, ids=lambda s: lbm.STORAGE_NAMES[s])
def test_small_lattice_without_transverse_corrections(storage):
    _compare(workloads.duct(9, 8, 7, (0.02, 0.01, 0.01), 0.9), storage, 1, (8,), no_n=True)


@pytest.mark.parametrize("storage", STORAGES, ids=lambda s: lbm.STORAGE_NAMES[s])
@pytest.mark.parametrize("spec", [workloads.duct(130, 97, 96, (0.04, 0.01, 0.01), 0.8),
                                  workloads.LatticeSpec(256, 105, 128, 0.9, {}, name="periodic_256x105x128")],
                         ids=lambda s: s.name)
def test_larger_lattices(spec, storage):
    _compare(spec, storage, 1, (5, 8, 3))


@pytest.mark.parametrize("chunk", [10, 14, 100])
@pytest.mark.parametrize("storage", ["f32", "f64", "f16sr"])
def test_single_jobs_of_a_batch(storage, chunk):
    specs = [workloads.duct(16, 16, 16, (0.03, 0.01, 0.0), 0.9), workloads.duct(40, 30, 20, (0.02, 0.01, 0.01), 0.8),
             workloads.duct(128, 96, 96, (0.04, 0.01, 0.01), 0.8)]
    steps = 2 * chunk
    b = lbm.lbm_batch_create(2 << 30, chunk, 4)
    try:
        lbm.lbm_batch_set_policy(b, lbm.LBM_BATCH_LARGE_IN_ORDER, 1 << 18)
        lbm.lbm_batch_set_lanes(b, 2)
        ids = [lbm.lbm_batch_submit(b, serving.job_for(s, storage, 0.0, steps)) for s in specs]
        while lbm.lbm_batch_run_chunk(b) != (0, 0):
            pass
        for jid, s in zip(ids, specs):
            rho, u = lbm.lbm_batch_result(b, jid, s.nodes)
            h = lbm.lbm_create(s.nx, s.ny, s.nz, s.tau, 1.0, None, serving.STORAGE[storage], torch.cuda.current_stream())
            serving.apply_bc(h, s)
            for _ in range(steps):
                lbm.lbm_step(h, 1)
            r, v = np.empty(s.nodes), np.empty(3 * s.nodes)
            lbm.lbm_moments(h, r, v)
            lbm.lbm_destroy(h)
            np.testing.assert_array_equal(rho, r)
            np.testing.assert_array_equal(u, v)
    finally:
        lbm.lbm_batch_destroy(b)


@pytest.mark.parametrize("chunk", [4, 10, 50])
@pytest.mark.parametrize("shape", [(256, 256, 0), (128, 1024, 64)], ids=["a-workgroup-per-tile", "persistent"])
def test_shared_chunks(chunk, shape):
    """A lockstep batch whose larger FP32 and FP64 jobs make passes beside
    jobs that do not (narrow, 16-bit), the convergence measure included."""
    items = [(workloads.duct(250, 120, 100, (0.03, 0.01, 0.0), 0.9), "f32"),
             (workloads.duct(33, 91, 20, (0.02, 0.01, 0.01), 0.8), "f32"),
             (workloads.duct(200, 100, 60, (0.04, 0.01, 0.01), 0.8), "f64"),
             (workloads.duct(130, 70, 64, (0.02, -0.01, 0.01), 1.1), "f64"),
             (workloads.duct(64, 20, 20, (0.03, 0.0, 0.01), 0.9), "f16sr")]
    steps = 2 * chunk
    got = []
    for one_step in (False, True):
        b = lbm.lbm_batch_create(2 << 30, chunk, 8)
        try:
            if one_step:
                lbm.lbm_batch_set_steps_per_pass(b, 1, 0)
            lbm.lbm_batch_set_shape(b, *shape)
            ids = [lbm.lbm_batch_submit(b, serving.job_for(s, st, 0.0, steps)) for s, st in items]
            while lbm.lbm_batch_run_chunk(b) != (0, 0):
                pass
            got.append([(lbm.lbm_batch_poll(b, i).delta, *lbm.lbm_batch_result(b, i, s.nodes))
                        for i, (s, _) in zip(ids, items)])
        finally:
            lbm.lbm_batch_destroy(b)
    for (s, st), x, y in zip(items, *got):
        assert x[0] == y[0], (s.name, st)
        np.testing.assert_array_equal(x[1], y[1], err_msg=s.name)
        np.testing.assert_array_equal(x[2], y[2], err_msg=s.name)
