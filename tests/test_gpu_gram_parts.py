"""Centre moves and matvecs at m = 126 on a 6 x 6 lattice, where the free range of
the effective-operator update's grams (126 x 126) is just above a whole number of
parts: against the oracle, 1e-12 relative as at the other ragged legs."""
import numpy as np
import pytest

from problems import make_problem
from tests.gpu_util import gpu_matvec, make_pair, move_both, rel

pytestmark = pytest.mark.gpu


def test_matvec_after_moves_at_126():
    a, o = make_pair(make_problem("ragged", 6, "ising", 126, 226, 6))
    a.validate()
    rng = np.random.default_rng(126)
    sizes = [int(np.prod(t.shape)) for t in o.T]
    for n in sorted(range(o.tree.n_nodes), key=lambda n: -sizes[n])[:2] + [o.tree.root]:
        print(f"node {n} {o.T[n].shape}", flush=True)
        move_both(a, o, n)
        x = rng.standard_normal(o.T[n].shape)
        assert rel(gpu_matvec(a, n, x), o.matvec(n, x)) < 1e-12, (n, x.shape)
    a.close()
