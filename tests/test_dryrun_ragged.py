"""Work lists of instances whose legs are no multiple of 16, checked on the host:
every operand, partial output, conversion and gram range of every node lies inside
its allocation, for the tile counts around the edges of the matrix-core kernels
(16, 32, 64, 128), above them, and on a lattice whose side gives uneven trees."""
import pytest

from paper_2507_21236_amd import ATTN_DRYRUN, AttnHandle
from problems import make_problem


@pytest.mark.parametrize("L,model,m", [(4, "heisenberg_tri", 7), (5, "ising", 15), (5, "ising", 17), (5, "ising", 31),
                                       (5, "ising", 33), (6, "heisenberg_tri", 50), (5, "ising", 63), (5, "ising", 65),
                                       (5, "ising", 100), (5, "ising", 127), (5, "ising", 130), (8, "ising", 48)])
def test_ragged_work_lists_in_bounds(L, model, m):
    a = AttnHandle(make_problem("ragged", L, model, m, m, 4), flags=ATTN_DRYRUN)
    a.validate()
    a.close()
