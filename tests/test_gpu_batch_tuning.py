"""What a batch makes of its jobs without being asked: the shape it tunes or takes
over, the padding of rows, passes in shared chunks, grouped steps on lanes; the
same bits each way."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0811_4593_amd import lbm, serving, workloads  # noqa: E402


def _trial_steps(nz):
    """Steps that tuning a batch of an FP64 duct of nz planes, whose boxes fill
    the device, and a small FP16 one takes: none when it finds a result."""
    b = lbm.lbm_batch_create(3 << 30, 100, 2)
    try:
        i = lbm.lbm_batch_submit(b, serving.job_for(workloads.duct(128, 98, nz, (0.03, 0.01, 0.0), 0.9), "f64", 0.0, 1000))
        lbm.lbm_batch_submit(b, serving.job_for(workloads.duct(20, 18, 16, (0.03, 0.01, 0.0), 0.9), "f16dev", 0.0, 1000))
        lbm.lbm_batch_autotune(b, 2)
        return lbm.lbm_batch_poll(b, i).steps
    finally:
        lbm.lbm_batch_destroy(b)


def test_sizes_of_one_mix_are_tuned_separately():
    # 3.2 and 6.4 million nodes: 2^22 and 2^23
    assert _trial_steps(256) > 0
    assert _trial_steps(512) > 0
    assert _trial_steps(256) == 0 and _trial_steps(512) == 0


def _flat_bytes(s):
    """Memory of an FP64 job with its populations one after another, without padded rows."""
    up = lambda n, m: (n + m - 1) // m * m  # noqa: E731
    return 2 * up(19 * up(s.nodes, 64) * 8, 256) + up(12 * s.nodes, 256)


def test_a_job_fits_the_budget_without_the_padding_of_passes():
    """Rows of 40 FP64 nodes take 48 with padding: a budget for the unpadded job
    takes it, and one job and a half at a time do not keep the second waiting."""
    s = workloads.duct(40, 70, 64, (0.03, 0.01, 0.0), 0.9)
    fields = []
    for budget, count in ((4 * _flat_bytes(s), 2), (_flat_bytes(s) + 4096, 1), (int(2.15 * _flat_bytes(s)), 2)):
        b = lbm.lbm_batch_create(budget, 20, 4)
        try:
            ids = [lbm.lbm_batch_submit(b, serving.job_for(s, "f64", 0.0, 40)) for _ in range(count)]
            assert lbm.lbm_batch_run_chunk(b) == (count, 0)
            while lbm.lbm_batch_run_chunk(b) != (0, 0):
                pass
            fields += [lbm.lbm_batch_result(b, i, s.nodes) for i in ids]
        finally:
            lbm.lbm_batch_destroy(b)
    for rho, u in fields[1:]:
        assert (rho == fields[0][0]).all() and (u == fields[0][1]).all()


def _padded(jobs, chunk, lanes=1):
    """Which of the queued FP64 ducts (extents) a batch stores with padded rows."""
    b = lbm.lbm_batch_create(4 << 30, chunk, len(jobs))
    try:
        lbm.lbm_batch_set_lanes(b, lanes)
        specs = [workloads.duct(*d, (0.03, 0.01, 0.0), 0.9) for d in jobs]
        for s in specs:
            lbm.lbm_batch_submit(b, serving.job_for(s, "f64", 0.0, 1000))
        lbm.lbm_batch_run_chunk(b)
        return lbm.lbm_batch_memory(b)[0] > sum(_flat_bytes(s) for s in specs)
    finally:
        lbm.lbm_batch_destroy(b)


@pytest.mark.parametrize("chunk, padded", [(2, False), (4, False), (6, True), (100, True)])
def test_padding_only_where_a_chunk_makes_passes(chunk, padded):
    """A chunk of up to four steps has no room for a pair of passes before its
    last step, so its jobs keep their unpadded rows."""
    assert _padded([(40, 70, 64)] * 25, chunk) == padded


@pytest.mark.parametrize("lanes", [1, 4])
@pytest.mark.parametrize("jobs, padded", [
    ([(40, 70, 64)] * 5, False),     # 200 boxes: less than one per compute unit
    ([(40, 70, 64)] * 8, False),     # 320 boxes, the second wave nearly empty
    ([(40, 70, 64)] * 100, True),    # thousands of boxes
    ([(40, 70, 64)], False),         # alone, steps not grouped
    ([(100, 100, 100)], True),       # alone, by passes
    ([(40, 28, 32)], True),          # alone, by blocks of steps
], ids=["few", "empty-wave", "many", "alone", "alone-passes", "alone-blocks"])
def test_padding_only_where_steps_are_grouped(jobs, padded, lanes):
    if len(jobs) == 100:
        jobs = [(40, 70, 16)] * 300 if lanes == 4 else jobs[:25]  # 3000 and 1000 boxes
    assert _padded(jobs, 100, lanes) == padded


def _launches(b):
    """Launches of several steps so far: multi-lattice passes, and those of chunks of one job."""
    out = ctypes.c_longlong(), ctypes.c_longlong()
    ctypes.CDLL(lbm.LIB_PATH).lbm_internal_batch_launches(ctypes.c_void_p(b), *map(ctypes.byref, out))
    return tuple(v.value for v in out)


def _passes(b):
    return _launches(b)[0]


# (each mix of forms is tuned once in a process)
@pytest.mark.parametrize("trial, small", [(2, ["f16sr"]), (4, ["f16dev"]), (6, ["f16sr", "f16dev"]), (16, [])])
def test_tuning_times_the_passes_of_a_default_batch(trial, small):
    """Of the trial steps the jobs that make passes in a chunk make them too;
    the number of steps and the state do not depend on that."""
    items = [(workloads.duct(128, 98, 113, (0.03, 0.01, 0.0), 0.9), "f64"),
             (workloads.duct(127, 98, 100, (0.02, 0.01, 0.01), 0.8), "f64"),
             (workloads.duct(33, 20, 30, (0.02, 0.01, 0.01), 0.8), "f64"),
             (workloads.duct(256, 156, 160, (0.03, 0.0, 0.01), 0.9), "f32")]
    items += [(workloads.duct(33, 20, 22, (0.02, 0.01, 0.01), 0.8), st) for st in small]
    got = []
    for tune in (True, False):
        steps = 6 * (2 + trial)
        b = lbm.lbm_batch_create(4 << 30, 6 if tune else steps + 6, 8)
        try:
            if not tune:
                lbm.lbm_batch_set_steps_per_pass(b, 1)
            ids = [lbm.lbm_batch_submit(b, serving.job_for(s, st, 0.0, steps + 6)) for s, st in items]
            if tune:
                lbm.lbm_batch_autotune(b, trial)
                assert [lbm.lbm_batch_poll(b, i).steps for i in ids] == [steps] * len(items)
                assert (_passes(b) > 0) == (trial >= 4)
            while lbm.lbm_batch_run_chunk(b) != (0, 0):
                pass
            got.append([lbm.lbm_batch_result(b, i, s.nodes) for i, (s, _) in zip(ids, items)])
        finally:
            lbm.lbm_batch_destroy(b)
    for (s, st), (rho, u), (r, v) in zip(items, *got):
        assert (rho == r).all() and (u == v).all(), (s.name, st)


@pytest.mark.parametrize("chunk", [6, 10, 50])
@pytest.mark.parametrize("shape", [(256, 256, 0), (128, 1024, 64)], ids=["a-workgroup-per-tile", "persistent"])
def test_shared_chunks_by_passes(chunk, shape):
    """A lockstep batch whose larger jobs make passes (asserted) beside jobs that
    do not, the convergence measure included, against single steps."""
    items = [(workloads.duct(250, 130, 112, (0.03, 0.01, 0.0), 0.9), "f32"),
             (workloads.duct(128, 117, 160, (0.03, 0.01, 0.0), 0.9), "f32"),
             (workloads.duct(33, 91, 20, (0.02, 0.01, 0.01), 0.8), "f32"),
             (workloads.duct(127, 98, 100, (0.04, 0.01, 0.01), 0.8), "f64"),
             (workloads.duct(128, 97, 113, (0.02, -0.01, 0.01), 1.1), "f64"),
             (workloads.duct(64, 20, 20, (0.03, 0.0, 0.01), 0.9), "f16sr")]
    got = []
    for one_step in (False, True):
        b = lbm.lbm_batch_create(4 << 30, chunk, 8)
        try:
            if one_step:
                lbm.lbm_batch_set_steps_per_pass(b, 1, 0)
            lbm.lbm_batch_set_shape(b, *shape)
            ids = [lbm.lbm_batch_submit(b, serving.job_for(s, st, 0.0, 2 * chunk)) for s, st in items]
            while lbm.lbm_batch_run_chunk(b) != (0, 0):
                pass
            # one captured chunk: the passes of two storage forms
            assert _passes(b) == (0 if one_step else 2 * (((chunk - 1) // 2) & ~1))
            got.append([(lbm.lbm_batch_poll(b, i).delta, *lbm.lbm_batch_result(b, i, s.nodes))
                        for i, (s, _) in zip(ids, items)])
        finally:
            lbm.lbm_batch_destroy(b)
    for (s, st), x, y in zip(items, *got):
        assert x[0] == y[0] and (x[1] == y[1]).all() and (x[2] == y[2]).all(), (s.name, st)


LARGE, SMALL = workloads.duct(128, 96, 96, (0.03, 0.01, 0.0), 0.9), workloads.duct(30, 30, 30, (0.02, 0.01, 0.0), 0.9)


def _grouped(policy, jobs, rounds=1):
    """Launches of several steps that chunks of one job make in `rounds` rounds
    of a batch with four lanes, and the fields of the jobs at their end."""
    b = lbm.lbm_batch_create(1 << 30, 20, 8)
    try:
        lbm.lbm_batch_set_policy(b, policy, 1 << 18)
        lbm.lbm_batch_set_lanes(b, 4)
        ids = [lbm.lbm_batch_submit(b, serving.job_for(s, st, 0.0, n)) for s, st, n in jobs]
        for _ in range(rounds):
            lbm.lbm_batch_run_chunk(b)
        n = _launches(b)[1]
        while lbm.lbm_batch_run_chunk(b) != (0, 0):
            pass
        return n, _launches(b)[1], [lbm.lbm_batch_result(b, i, s.nodes) for i, (s, _, _) in zip(ids, jobs)]
    finally:
        lbm.lbm_batch_destroy(b)


def test_lanes_group_steps_only_alike():
    """Alone, a job groups its steps (20: 8 passes or 8 blocks of two); beside a job
    whose launches are of another kind it does not, in whichever order they
    come; beside one of its own kind it does; the bits are the same."""
    order = lbm.LBM_BATCH_LARGE_IN_ORDER
    n, _, alone = _grouped(order, [(LARGE, "f64", 20)])
    assert n == 8
    n, _, small = _grouped(order, [(SMALL, "f32", 20)])
    assert n == 8
    for jobs in ([(LARGE, "f64", 20), (SMALL, "f32", 20)], [(SMALL, "f32", 20), (LARGE, "f64", 20)]):
        n, _, both = _grouped(order, jobs)
        assert n == 0
        for (s, _, _), (rho, u) in zip(jobs, both):
            r, v = (alone if s is LARGE else small)[0]
            assert (rho == r).all() and (u == v).all()
    # FP16 makes single sweeps at this size: a small job beside it does not make blocks
    assert _grouped(order, [(LARGE, "f16sr", 20), (SMALL, "f32", 20)])[0] == 0
    assert _grouped(order, [(SMALL, "f32", 20), (SMALL, "f64", 20)])[0] == 16
    assert _grouped(lbm.LBM_BATCH_SHORTEST_FIRST, [(LARGE, "f64", 20), (LARGE, "f32", 20)])[0] == 16
    # the large job goes back to passes when the small one has ended
    n, total, _ = _grouped(order, [(LARGE, "f64", 200), (SMALL, "f32", 20)])
    assert n == 0 and total >= 8 * 7
