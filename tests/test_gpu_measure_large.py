"""Products that meet at one large node (8 x 8, m = 128: 128^3 entries, 112 operator
images on either side), more than the engine stacks at once: all pairs in blocks of
rows and columns, and a few hundred pairs in groups, with work lists that fill the
upload stage more than once.  Reference: the same contraction in FP64 with torch,
one image at a time.  Tolerance 1e-12 of the largest value: unit roundoff times a
serial run of at most a few thousand summands.  After each call the handle keeps at
most two workspaces of 256 MB."""
import numpy as np
import pytest

from problems import make_problem
from tests.gpu_util import make_pair

pytestmark = pytest.mark.gpu


def _image(T, children, child, site, op):
    """The operator on one site carried up to the link above `child` (None: not below it)."""
    import torch
    if child[0] == "s":
        return op if child[1] == site else None
    t = T[child[1]]
    left, right = (_image(T, children, c, site, op) for c in children[child[1]])
    if left is None and right is None:
        return None
    d0, d1, d2 = t.shape
    if left is not None:
        x = left @ t.reshape(d0, d1 * d2)
    else:
        x = torch.matmul(right, t)
    return t.reshape(d0 * d1, d2).T @ x.reshape(d0 * d1, d2)


def test_products_meeting_at_a_large_node():
    import torch
    p = make_problem("large", 8, "ising", 128, 7, 8)
    a, o = make_pair(p)
    assert a.center == o.tree.root == o.center
    ch = o.tree.children
    n = ch[o.tree.root][0][1]   # 32 sites below it, 16 on either side
    assert o.T[n].shape == (128, 128, 128)

    def sites_below(child):
        return [child[1]] if child[0] == "s" else [s for c in ch[child[1]] for s in sites_below(c)]

    rng = np.random.default_rng(3)
    sides = []
    for c in ch[n]:
        sites = sites_below(c)
        assert len(sites) == 16
        sides.append([(s, rng.standard_normal((2, 2))) for s in sites for _ in range(7)])
    L, R = sides

    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    print("all pairs", flush=True)
    got = np.array(a.expect_products([[x, y] for x in L for y in R])).reshape(len(L), len(R))
    assert free0 - torch.cuda.mem_get_info()[0] <= 520 << 20
    pairs = [(int(i), int(j)) for i, j in zip(np.r_[np.arange(112), rng.integers(0, 112, 188)],
                                              np.r_[rng.permutation(112), rng.integers(0, 112, 188)])]
    print("single pairs", flush=True)
    few = np.array(a.expect_products([[L[i], R[j]] for i, j in pairs]))
    assert free0 - torch.cuda.mem_get_info()[0] <= 520 << 20
    print("all pairs again", flush=True)
    again = np.array(a.expect_products([[x, y] for x in L for y in R])).reshape(len(L), len(R))
    a.close()
    assert np.array_equal(got, again)

    T = {k: torch.from_numpy(np.ascontiguousarray(t)).cuda() for k, t in enumerate(o.T)}
    root = T[o.tree.root][:, :, 0]
    t = T[n]
    w = torch.matmul(t.reshape(-1, 128), root @ root.T).reshape(128, 128, 128)   # the root on the link above
    U = torch.stack([(_image(T, ch, ch[n][0], s, torch.from_numpy(x).cuda()).T @ t.reshape(128, -1)).reshape(-1)
                     for s, x in L])
    want = np.empty((len(L), len(R)))
    for j, (s, x) in enumerate(R):
        v = torch.matmul(_image(T, ch, ch[n][1], s, torch.from_numpy(x).cuda()), w).reshape(-1)
        want[:, j] = torch.mv(U, v).cpu().numpy()
    top = np.abs(want).max()
    assert np.abs(got - want).max() <= 1e-12 * top, np.abs(got - want).max() / top
    ref = np.array([want[i, j] for i, j in pairs])
    assert np.abs(few - ref).max() <= 1e-12 * top, np.abs(few - ref).max() / top
