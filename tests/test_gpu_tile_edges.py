"""Sizes at the edges of the work splits, through the C interface against the
oracle.  Solves: nodes of m^3 entries on both sides of the one-workgroup solver's
end (9 and 10: 729 and 1000 entries, the split between its two forms) and of the
partial sums' chunk sizes (12/13 and 16/17, where an entry's sum passes from 64
to 32 and from 32 to 16 threads); energies per site to 1e-10 as for every other
solve.  Observables: links around the tiles of 32 and 64 of their products and
results on both sides of them, to 1e-12 (values of order 1, unit roundoff
1.1e-16 times the few thousand summands of an entry)."""
import numpy as np
import pytest

from oracle.measure import measure, product_expectation
from problems import make_problem
from problems.models import PX, PZ
from tests.gpu_util import make_pair, move_both, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [9, 10, 12, 13, 16, 17])
def test_solves_at_the_edges_of_the_splits(m):
    p = make_problem("edges", 5, "ising", m, 30 + m, 6)
    a, o = make_pair(p)
    for _ in range(2):
        got, _ = a.sweep(1)
        want = o.sweep()
        assert abs(got[-1] - want) / p.n_sites < 1e-10, (m, got, want)
    a.close()


@pytest.mark.parametrize("m", [7, 16, 31, 32, 33, 65])
def test_observables_at_the_edges_of_the_tiles(m):
    p = make_problem("edges", 5, "ising", m, 60 + m, 6)
    a, o = make_pair(p)
    rng = np.random.default_rng(m)
    items = [[(int(s), rng.standard_normal((2, 2))) for s in rng.choice(p.n_sites, k, replace=False)]
             for k in (1, 2, 3, 4)]
    for it, g in zip(items, a.expect_products(items)):
        want = product_expectation(o.tree, o.T, dict(it))
        assert abs(g - want) <= 1e-12 * max(1.0, abs(want)), (m, it, g, want)
    C = a.correlation(PZ, PX)
    pairs = [tuple(ab) for ab in p.de_sites[:2]] + [tuple(int(x) for x in rng.choice(p.n_sites, 2, replace=False))
                                                    for _ in range(10)]
    for i, j in pairs:
        want = measure(o.tree, o.T, [i, j], [PZ, PX], p.de_sites, p.de_u)
        assert abs(C[i, j] - want) <= 1e-12, (m, i, j, C[i, j], want)
    a.close()


@pytest.mark.parametrize("m", [32, 64, 96, 128])
def test_split_bf16_matvecs_at_every_chunk_count(m):
    import torch
    from paper_2507_21236_amd import ATTN_BF16X2
    p = make_problem("edges", 5, "ising", m, 90 + m, 6)
    a, o = make_pair(p)
    rng = np.random.default_rng(m)
    sizes = [int(np.prod(t.shape)) for t in o.T]
    for n in sorted(range(o.tree.n_nodes), key=lambda n: -sizes[n])[:3] + [o.tree.root]:
        move_both(a, o, n)
        x = torch.from_numpy(rng.standard_normal(o.T[n].shape)).to("cuda", torch.float32)
        y = torch.empty_like(x)
        a.heff_apply(n, x, y, dtype=ATTN_BF16X2)
        torch.cuda.synchronize()
        assert rel(y.double().cpu().numpy(), o.matvec(n, x.double().cpu().numpy())) < 1e-4, (m, n, x.shape)
    a.close()
