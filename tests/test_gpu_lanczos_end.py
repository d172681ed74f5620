"""Eigensolves in a two-dimensional invariant subspace with <H> = 0, where every
diagonal Lanczos coefficient is of rounding's size and the run can only end by what
is left of the residual: the value returned is the Rayleigh quotient of the tensor
returned, which is normalised, to 1e-12 (of the spectrum's size 1)."""
import dataclasses

import numpy as np
import pytest

from problems import make_problem
from problems.models import PX
from tests.gpu_util import gpu_matvec, make_pair, move_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [12, 16, 33])
def test_value_is_the_rayleigh_quotient(m):
    from paper_2507_21236_amd import AttnHandle
    base = make_problem("end", 5, "ising", m, 200 + m, 0)
    base = dataclasses.replace(base, de_sites=[], de_u=np.zeros((0, 4, 4)))
    shapes = [r.shape for r in base.raw_tensors]
    n = max(range(len(shapes)), key=lambda k: np.prod(shapes[k]))
    p = dataclasses.replace(base, terms=[((3,), [PX], 1.0)])
    a, o = make_pair(p)
    move_both(a, o, n)
    # the term acts on one leg: its matrix from slices of unit vectors
    dims = o.T[n].shape
    x = np.random.default_rng(m).standard_normal(dims)
    y = gpu_matvec(a, n, x)
    legs = [_leg_matrix(a, n, dims, l) for l in range(3)]   # a multiple of 1 where the term does not act
    leg = max(range(3), key=lambda l: np.linalg.norm(legs[l] - np.diag(np.diag(legs[l]))))
    A = legs[leg]
    assert np.allclose(np.moveaxis(np.tensordot(A, x, axes=(1, leg)), 0, leg), y, atol=1e-12)
    lam, U = np.linalg.eigh((A + A.T) / 2)
    a.close()
    # shifted so that the two outer eigenvalues are opposite, started with equal weights on both
    shift = -(lam[0] + lam[-1]) / 2
    q = dataclasses.replace(p, terms=p.terms + [((7,), [np.eye(2)], float(shift))])
    b = AttnHandle(q)
    b.init_state()
    b.move_center(n)
    rest = np.random.default_rng(m + 1).standard_normal([d for l, d in enumerate(dims) if l != leg])
    v = np.moveaxis(np.multiply.outer(U[:, 0] + U[:, -1], rest), 0, leg)
    b.set_tensor(n, v / np.linalg.norm(v))
    theta, _ = b.eigsolve(n)
    t = b.get_tensor(n)
    hv = gpu_matvec(b, n, t)
    print(f"m {m}: theta {theta:.15f}, half gap {(lam[-1] - lam[0]) / 2:.15f}")
    assert abs(np.linalg.norm(t) - 1) < 1e-12
    assert abs(np.vdot(t, hv) - theta) < 1e-12
    assert abs(theta + (lam[-1] - lam[0]) / 2) < 1e-12   # the lowest value of the shifted operator
    b.close()


def _leg_matrix(a, n, dims, leg):
    """H restricted to leg `leg` at the first index of the other two (exact when H acts on it alone)."""
    M = np.zeros((dims[leg], dims[leg]))
    for i in range(dims[leg]):
        e = np.zeros(dims)
        at = [0, 0, 0]
        at[leg] = i
        e[tuple(at)] = 1.0
        y = gpu_matvec(a, n, e)
        at[leg] = slice(None)
        M[:, i] = y[tuple(at)]
    return M
