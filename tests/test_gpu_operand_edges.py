"""Ragged legs read nothing past the end of their operands: mode products and
sandwiches on operator blocks and tensors that lie in the middle of an allocation
full of NaN give finite results, equal to FP64 (FP32: to 1e-5) products of the same
operands.  The kernels pad K steps and tiles with zeros; memory behind a block is
usually finite, so a read past its end would not show elsewhere.  1e-12 and 1e-5
relative: unit roundoff times a few hundred summands.  The same for slices of more
than four row strips that are cut into work units of four."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GUARD = 1 << 15   # elements of NaN on both sides: more than two tiles of the widest block


class Job(ctypes.Structure):
    _fields_ = [("A", ctypes.c_void_p), ("x", ctypes.c_void_p), ("coef", ctypes.c_double)]


class MPTask(ctypes.Structure):
    _fields_ = [("out", ctypes.c_void_p), ("d", ctypes.c_int32 * 3), ("j", ctypes.c_int32), ("job0", ctypes.c_int32),
                ("njob", ctypes.c_int32), ("accumulate", ctypes.c_int32), ("pad", ctypes.c_int32)]


class SWTask(ctypes.Structure):
    _fields_ = [("x", ctypes.c_void_p), ("y", ctypes.c_void_p), ("xs_slice", ctypes.c_int64),
                ("xs_row", ctypes.c_int64), ("ys_slice", ctypes.c_int64), ("ys_row", ctypes.c_int64),
                ("ma", ctypes.c_int32), ("mb", ctypes.c_int32), ("item0", ctypes.c_int32), ("nitem", ctypes.c_int32),
                ("accumulate", ctypes.c_int32), ("pad", ctypes.c_int32)]


def _guarded(x, dtype):
    """(allocation, address) of a copy of x between two runs of NaN."""
    import torch
    n = x.size
    t = torch.full((n + 2 * GUARD,), float("nan"), dtype=dtype, device="cuda")
    t[GUARD:GUARD + n] = torch.from_numpy(np.ascontiguousarray(x).ravel()).to("cuda", dtype)
    return t, t.data_ptr() + GUARD * t.element_size()


def _upload(*items):
    """Device copy of structures or arrays: (tensor, address)."""
    import torch
    raw = b"".join(bytes(i) if isinstance(i, ctypes.Structure) else i.tobytes() for i in items)
    t = torch.frombuffer(bytearray(raw), dtype=torch.uint8).cuda()
    return t, t.data_ptr()


def _launch(name, *args):
    import torch
    from paper_2507_21236_amd import _lib
    torch.cuda.synchronize()
    assert getattr(_lib._lib, "_ZN4attn25prepare_kernel_attributesEv")() == 0
    assert getattr(_lib._lib, name)(*args) == 0
    torch.cuda.synchronize()


def _ptr(p):
    return ctypes.c_void_p(p)


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("mj", [9, 17, 31, 33, 50, 63, 65, 90, 100, 113, 127])
def test_mode_products_of_ragged_legs(mj, f32):
    import torch
    dt, esz = (torch.float32, 4) if f32 else (torch.float64, 8)
    rng = np.random.default_rng(mj)
    for j in range(3):
        d = [11, 13, 7]
        d[j] = mj
        A, x = rng.standard_normal((mj, mj)), rng.standard_normal(d)
        print(f"mode mj {mj} leg {j} f32 {f32}", flush=True)
        ta, pa = _guarded(A.T, dt)   # column-major blocks
        tx, px = _guarded(x, dt)
        to, po = _guarded(np.zeros(d), dt)
        tt = MPTask(po, (ctypes.c_int32 * 3)(*d), j, 0, 2, 0, 0)
        k1 = _upload(tt)
        k2 = _upload(Job(pa, px, 0.75), Job(pa, px, -0.25))
        nb = (x.size // mj + 63) // 64
        k3 = _upload(np.array([[0, f] for f in range(nb)], dtype=np.int32))
        _launch("_ZN4attn11launch_modeEiibPKNS_6MPTaskEPKNS_5MPJobEPK15HIP_vector_typeIiLj2EEiPKvP12ihipStream_t",
                int(f32), mj, True, _ptr(k1[1]), _ptr(k2[1]), _ptr(k3[1]), nb, None, None)
        got = to[GUARD:GUARD + x.size].double().cpu().numpy().reshape(d)
        want = 0.5 * np.moveaxis(np.tensordot(A, x, axes=(1, j)), 0, j)
        assert np.isfinite(got).all(), (mj, j)
        assert np.abs(got - want).max() <= (1e-5 if f32 else 1e-12) * np.abs(want).max(), (mj, j)
        assert torch.isnan(to[:GUARD]).all() and torch.isnan(to[GUARD + x.size:]).all(), (mj, j)


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("ma,mb", [(17, 17), (31, 33), (50, 50), (49, 64), (64, 50), (65, 65), (100, 90), (7, 100),
                                   (113, 97), (127, 127), (127, 17), (3, 127)])
def test_sandwiches_of_ragged_slices(ma, mb, f32):
    _sandwich(ma, mb, f32, 0)


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("ma,mb", [(65, 65), (80, 80), (96, 33), (100, 90), (112, 112), (127, 127), (128, 128), (128, 64)])
def test_slices_in_units_of_four_strips(ma, mb, f32):
    _sandwich(ma, mb, f32, 4)


def _sandwich(ma, mb, f32, strips):
    import torch
    dt = torch.float32 if f32 else torch.float64
    rng = np.random.default_rng(1000 * ma + mb)
    ns = 3
    A, B, x = rng.standard_normal((ma, ma)), rng.standard_normal((mb, mb)), rng.standard_normal((ns, ma, mb))
    print(f"sandwich {ma} x {mb} f32 {f32}", flush=True)
    ta, pa = _guarded(A.T, dt)
    tb, pb = _guarded(B.T, dt)
    tx, px = _guarded(x, dt)
    ty, py = _guarded(np.zeros_like(x), dt)
    # items without B first: 0.5 A X, then A X B^T and X B^T
    k2 = _upload(Job(pa, None, 0.5), Job(pa, pb, 1.0), Job(None, pb, -0.25))
    k1 = _upload(SWTask(px, py, ma * mb, mb, ma * mb, mb, ma, mb, 0, 3, 0, 0))
    units = [[0, s, st, 0] for s in range(ns) for st in range(0, -(-ma // 16), strips or 8)]
    k3 = _upload(np.array(units, dtype=np.int32))
    _launch("_ZN4attn15launch_sandwichEiiiPKNS_6SWTaskEPKNS_6SWItemEPK15HIP_vector_typeIiLj4EEiPKvP12ihipStream_tPKNS_5SWOutEi",
            int(f32), ma, mb, _ptr(k1[1]), _ptr(k2[1]), _ptr(k3[1]), len(units), None, None, None, strips)
    got = ty[GUARD:GUARD + x.size].double().cpu().numpy().reshape(x.shape)
    ax = np.einsum("ij,sjk->sik", A, x)
    want = 0.5 * ax + ax @ B.T - 0.25 * x @ B.T
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= (1e-5 if f32 else 1e-12) * np.abs(want).max()
    assert torch.isnan(ty[:GUARD]).all() and torch.isnan(ty[GUARD + x.size:]).all()
