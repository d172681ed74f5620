"""The choice between the staged and the persistent form of a batch (persistent = 2)
times the launches that a sweep makes: in FP64 the staged form ends in the sum fused
with its dots, the persistent one in dots of its own, as the recorded kernels of the
batch's creation show; and a batch that chose per step sweeps to the same bits."""
import numpy as np
import pytest

from problems import make_problem

pytestmark = pytest.mark.gpu


def _handles():
    from paper_2507_21236_amd import AttnHandle
    hs = [AttnHandle(make_problem(f"f{m}", 5, "ising", m, m, 6)) for m in (12, 17, 24)]
    for h in hs:
        h.init_state()
    return hs


def test_choice_times_the_launches_of_a_sweep():
    from torch.profiler import ProfilerActivity, profile
    from paper_2507_21236_amd import ATTN_F64, AttnBatch
    hs = _handles()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        b = AttnBatch(hs, precision=ATTN_F64, persistent=2)
    names = {e.key for e in prof.key_averages()}
    if not any("k_batch_matvec" in n for n in names):
        pytest.skip("the profiler recorded no kernels")
    assert any("k_reduce_dots_list" in n for n in names), names
    assert any("k_kdots" in n for n in names), names
    assert not any("k_reduce_list" in n for n in names), names
    got, _ = b.sweep(2)
    b.close()
    ref, _ = AttnBatch(_handles(), precision=ATTN_F64).sweep(2)
    assert np.array_equal(got, ref)
