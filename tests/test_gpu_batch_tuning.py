"""lbm_batch_autotune: a batch takes over the shape tuned for an earlier one only
if it holds the same kind of work (storage forms and how they step, resident
nodes to a power of two)."""
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
