"""Every observable call synchronises the device: work that the caller has in flight
on a stream of its own (which does not wait for the default stream, nor the other
way round) has ended when the call returns."""
import numpy as np
import pytest

from problems import make_problem
from problems.models import PZ

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("call", ["products", "measure", "correlation"])
def test_observables_wait_for_other_streams(call):
    import torch
    from paper_2507_21236_amd import AttnHandle
    a = AttnHandle(make_problem("sync", 4, "ising", 8, 5, 4))
    a.init_state()
    run = {"products": lambda: a.expect_products([[(0, PZ), (5, PZ)]]), "measure": lambda: a.measure([[(3, PZ)]]),
           "correlation": lambda: a.correlation(PZ, PZ)}[call]
    want = run()
    side = torch.cuda.Stream()
    x = torch.randn(8192, 8192, dtype=torch.float32, device="cuda") * 1e-3
    y = torch.empty_like(x)
    torch.mm(x, x, out=y)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(60):   # some tens of times the observable's own time
            torch.mm(x, x, out=y)
    got = run()
    assert side.query(), "the call returned with work in flight"
    assert np.array_equal(got, want)
    torch.cuda.synchronize()
    a.close()
