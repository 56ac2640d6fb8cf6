"""Tensor handles in unusual states: moved-from operands, operands and results
that share memory."""
import ctypes

import numpy as np
import pytest

from paper_2512_23917_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    from paper_2512_23917_amd import tci
    return tci


@pytest.fixture(scope="module")
def ctx(T):
    c = T.Context(0)
    yield c
    c.close()


def draw(shape, seed):
    return synth.complex_gaussian(synth.rng(41, seed), shape)


@pytest.mark.parametrize("side", [0, 1])
def test_moved_from_operand_is_refused(T, ctx, side):
    """A handle keeps its dimensions when its data is moved away; an update that gets it fails on the host."""
    ops = [[T.Tensor.from_numpy(ctx, draw(s, i), T.C128) for i in range(2)] for s in ((3, 2, 4), (4, 2, 3))]
    taken = ctypes.c_void_p()
    T._check(T.lib().tci_move(ctx.h, ctypes.byref(ops[side][1].h), ctypes.byref(taken)), "tci_move")
    p = T.update_params(chi_min=1, chi_max=4, direction=T.DIR_LEFT)
    with pytest.raises(T.TciError):
        T.two_site_update_batched(ctx, ops[0], ops[1], None, p)
    T._check(T.lib().tci_destroy(ctx.h, taken), "tci_destroy")
    # the context goes on
    out = T.two_site_update_batched(ctx, ops[0][:1], ops[1][:1], None, p) if side else None
    assert out is None or out[3][0].chi == 4


# up to 2^17 multiply-adds (one launch) and above, the result permuted and in its own order
@pytest.mark.parametrize("la,lb,lc,dims", [("ab", "bc", "ca", dict(a=3, b=4, c=5000)),
                                           ("ab", "bc", "ac", dict(a=3, b=4, c=5000)),
                                           ("ab", "bc", "ac", dict(a=3, b=70, c=5000)),
                                           ("ab", "bc", "ca", dict(a=3, b=70, c=5000))])
def test_result_grows_over_an_operand(T, ctx, la, lb, lc, dims):
    """The result's handle owns the memory that an operand wraps, and is too small: the operand is read first."""
    a, b = (draw([dims[x] for x in lab], 5 + i) for i, lab in enumerate((la, lb)))
    out, view, ptr = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_void_p()
    src, tb = T.Tensor.from_numpy(ctx, a, T.C128), T.Tensor.from_numpy(ctx, b, T.C128)
    L, shape = T.lib(), T._i64(a.shape)
    T._check(L.tci_copy(ctx.h, src.h, ctypes.byref(out)), "tci_copy")
    T._check(L.tci_data_ptr(ctx.h, out, ctypes.byref(ptr)), "tci_data_ptr")
    T._check(L.tci_wrap(ctx.h, T.C128, 2, shape, ptr, ctypes.byref(view)), "tci_wrap")
    T._check(L.tci_contract(ctx.h, view, T._i32([ord(x) for x in la]), 2, tb.h, T._i32([ord(x) for x in lb]), 2, out,
                            T._i32([ord(x) for x in lc]), 2), "tci_contract")
    ref = np.einsum(f"{la},{lb}->{lc}", a, b)
    got = T.Tensor.empty(ctx, T.C128, ref.size)
    T._check(L.tci_reshape(ctx.h, out, 2, T._i64(ref.shape), got.h), "tci_reshape")
    # sums of at most 70 products of values of order one
    assert np.abs(got.numpy() - ref).max() < 1e-13 * 70
    for h in (view, out):
        T._check(L.tci_destroy(ctx.h, h), "tci_destroy")


@pytest.mark.parametrize("shift", [1, 2, 4, 8])
def test_operands_at_any_address(T, ctx, shift):
    """Operands are copied before they are used, so a wrapped address may be any multiple of a byte."""
    arrs = [draw(s, 7 + i) for i, s in enumerate(((3, 2, 5), (5, 2, 3), (2, 2, 2, 2)))]
    ops, keep = [], []
    for a in arrs:
        buf = torch.zeros(a.nbytes + 16, dtype=torch.uint8, device="cuda")
        buf[shift:shift + a.nbytes] = torch.from_numpy(np.frombuffer(a.tobytes(), np.uint8).copy()).cuda()
        h = ctypes.c_void_p()
        T._check(T.lib().tci_wrap(ctx.h, T.C128, a.ndim, T._i64(a.shape), ctypes.c_void_p(buf.data_ptr() + shift),
                                  ctypes.byref(h)), "tci_wrap")
        ops.append(h)
        keep.append(buf)
    p = T.update_params(chi_min=1, chi_max=4, direction=T.DIR_LEFT)
    want = T.two_site_update_batched(ctx, *([T.Tensor.from_numpy(ctx, a, T.C128)] for a in arrs), p)
    out = [T.Tensor.empty(ctx, t, n) for t, n in ((T.C128, 24), (T.F64, 4), (T.C128, 24))]
    P, info = ctypes.c_void_p * 1, (T.UpdateInfo * 1)()
    T._check(T.lib().tci_two_site_update_batched(ctx.h, 1, *(P(h.value) for h in ops), ctypes.byref(p),
                                                 *(P(x.h.value) for x in out), info), "tci_two_site_update_batched")
    for x, y in zip(out, want[:3]):
        assert np.array_equal(x.numpy(), y[0].numpy())
    for h in ops:
        T._check(T.lib().tci_destroy(ctx.h, h), "tci_destroy")
