"""Bond dimensions that are no multiple of 16 (one and several tiles wide,
around the tile edges, up to the 128 limit of the matrix-core kernels) through
the C interface against the oracle: matvecs after centre moves, so that the
contraction, the effective-operator update, the QR and the absorption are all
checked at those legs.  Tolerances as for the whole-tile legs: 1e-12 relative
in FP64 and 1e-5 in FP32, whose unit roundoffs (1.1e-16, 6e-8) times the few
thousand summands of an entry stay below them."""
import numpy as np
import pytest

from problems import make_problem
from tests.gpu_util import gpu_matvec, make_pair, move_both, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [15, 17, 20, 31, 33, 50, 65, 100, 127])
def test_matvec_after_moves_at_ragged_legs(m):
    import torch
    from paper_2507_21236_amd import ATTN_F32
    p = make_problem("ragged", 5, "ising", m, 100 + m, 6)
    a, o = make_pair(p)
    rng = np.random.default_rng(m)
    sizes = [int(np.prod(t.shape)) for t in o.T]
    heavy = sorted(range(o.tree.n_nodes), key=lambda n: -sizes[n])
    for n in heavy[:3] + [0, o.tree.root]:
        move_both(a, o, n)
        x = rng.standard_normal(o.T[n].shape)
        want = o.matvec(n, x)
        assert rel(gpu_matvec(a, n, x), want) < 1e-12, (n, x.shape)
        x32 = torch.from_numpy(x).cuda().float()
        y32 = torch.empty_like(x32)
        a.heff_apply(n, x32, y32, dtype=ATTN_F32)
        torch.cuda.synchronize()
        assert rel(y32.double().cpu().numpy(), want) < 1e-5, (n, x.shape)
    a.close()


def test_batch_of_ragged_instances_matches_single_handles():
    """The batched launches share the tile bodies: the same energies bit for bit."""
    from paper_2507_21236_amd import ATTN_F64, AttnBatch, AttnHandle
    probs = [make_problem(f"r{m}", 5, "ising", m, m, 6) for m in (17, 24, 40, 63)]
    hs = [AttnHandle(p) for p in probs]
    for h in hs:
        h.init_state()
    got, _ = AttnBatch(hs, precision=ATTN_F64).sweep(2)
    for k, p in enumerate(probs):
        s = AttnHandle(p)
        s.init_state()
        want, _ = s.sweep(2)
        assert np.array_equal(got[k], want), (p.m, got[k], want)
