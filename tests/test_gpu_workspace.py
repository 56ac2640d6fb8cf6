"""Calls on workspace that holds NaN: memory of an allocator comes with the bits
of its last use, and a result may depend on none of them.  0xFF bytes are a NaN
in every floating type and -1 in every integer type."""
import ctypes

import numpy as np
import pytest

from paper_2512_23917_amd import synth
from gpu_util import isometry_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
U64 = 2.0 ** -53
WORKSPACE = 256 << 20    # workspace is requested in chunks of at least this size


@pytest.fixture(scope="module")
def T():
    from paper_2512_23917_amd import tci
    return tci


class Memory:
    """A context whose memory is filled with one byte, and filled again on request."""

    def __init__(self, T, byte):
        self.live, self.byte = {}, byte

        def alloc(n, s):
            x = torch.full((int(n),), byte, dtype=torch.uint8, device="cuda")
            torch.cuda.synchronize()
            self.live[x.data_ptr()] = x
            return x.data_ptr()

        self.ctx = T.Context(0, allocator=(alloc, lambda p, n, s: self.live.pop(p)))

    def refill(self):
        torch.cuda.synchronize()
        for x in self.live.values():
            if x.numel() >= WORKSPACE:
                x.fill_(self.byte)
        torch.cuda.synchronize()
        return self.ctx


@pytest.fixture(scope="module")
def poisoned(T):
    m = Memory(T, 0xFF)
    yield m
    m.ctx.close()


def draw(shape, complex_, seed):
    g = synth.rng(37, seed)
    return synth.complex_gaussian(g, shape) if complex_ else synth.real_gaussian(g, shape)


# 192 complex / 320 real: all columns on chip; one, two and 32 columns before them, several panels, a first band that
# is left behind
@pytest.mark.parametrize("complex_,n", [(True, 192), (True, 193), (True, 194), (True, 225), (True, 385), (True, 500),
                                        (False, 320), (False, 321), (False, 322), (False, 353), (False, 385),
                                        (False, 500)])
def test_decompositions(T, poisoned, complex_, n):
    """Backward stable eigensolver: n u ||A|| on its values; the Gram route leaves that of the largest square on the
    squared singular values."""
    code = T.C128 if complex_ else T.F64
    a = draw((n, n), complex_, n)
    h = (a + a.conj().T) / 2
    tol = (8 * n + 64) * U64
    ctx = poisoned.refill()
    w, v = (x.numpy() for x in T.eigh(ctx, T.Tensor.from_numpy(ctx, h, code)))
    ref = np.linalg.eigvalsh(h)
    scale = np.abs(ref).max()
    assert np.abs(w - ref).max() < tol * scale and np.abs(h @ v - v * w).max() < tol * scale
    ctx = poisoned.refill()
    assert np.abs(T.eigvalsh(ctx, T.Tensor.from_numpy(ctx, h, code)).numpy() - ref).max() < tol * scale
    ctx = poisoned.refill()
    u, s, vh, _ = T.trunc_svd(ctx, T.Tensor.from_numpy(ctx, a, code), 1, 1, n // 2)
    sr = np.linalg.svd(a, compute_uv=False)
    assert np.abs(s.numpy() ** 2 - sr[:n // 2] ** 2).max() < tol * sr[0] ** 2
    assert isometry_err(u.numpy()) < tol and isometry_err(vh.numpy(), False) < tol
    chi = (n + 1) // 2
    x, y = draw((chi, 2, 9), complex_, n + 1), draw((9, 2, chi), complex_, n + 2)
    p = T.update_params(chi_min=1, chi_max=9, direction=T.DIR_LEFT, precision=T.PREC_FP64)
    ctx = poisoned.refill()
    ao, so, bo, _ = T.two_site_update_batched(ctx, [T.Tensor.from_numpy(ctx, x, code)],
                                              [T.Tensor.from_numpy(ctx, y, code)], None, p)
    theta = np.einsum("asm,mtb->astb", x, y)
    theta /= np.linalg.norm(theta)
    assert np.abs(np.einsum("asm,mtb->astb", ao[0].numpy(), bo[0].numpy()) - theta).max() < 64 * tol


def _calls(T):
    """name -> call of a context that returns arrays."""
    from paper_2512_23917_amd import sketch_train
    d, f = (lambda *s: draw(s, True, sum(s))), (lambda *s: draw(s, False, sum(s)))
    lo = lambda x: x.astype(np.complex64)  # noqa: E731
    t = T.Tensor.from_numpy
    w = synth.heisenberg_mpo()

    def env(c, chi, code):
        e = d(chi, 5, chi)
        e[:, 2] = e[:, 1].conj().T
        for k in (0, 3, 4):
            e[:, k] = (e[:, k] + e[:, k].conj().T) / 2
        return t(c, e if code == T.C128 else lo(e), code)

    def matvec(prec):
        def go(c):
            c.set_precision(prec)
            return [T.heff_matvec(c, env(c, 37, T.C64), t(c, lo(w), T.C64), t(c, lo(w), T.C64), env(c, 41, T.C64),
                                  t(c, lo(d(37, 2, 2, 41)), T.C64))]
        return go

    def lanczos(c):
        th = t(c, d(20, 2, 2, 24), T.C128)
        T.lanczos_ground(c, env(c, 20, T.C128), t(c, w, T.C128), t(c, w, T.C128), env(c, 24, T.C128), th, 12)
        p = T.update_params(chi_min=1, chi_max=18, direction=T.DIR_RIGHT, precision=T.PREC_FP64)
        a, s, b, _ = T.split_batched(c, [th], p)
        return [th, s[0]]

    def sketch(mode):
        def go(c):
            g = synth.rng(5, 3)
            s = [synth.power_spectrum(300, x) for x in (1.2, 2.0, 2.9)]
            ab = [synth.two_site_blocks_from_spectrum(g, 150, 2, x) for x in s]
            p = T.update_params(chi_min=1, chi_max=150, target_trunc_err=1e-8, direction=T.DIR_LEFT,
                                precision=T.PREC_FP32, svd_mode=mode, power_iters=2, seed=1)
            if mode == T.SVD_RANDOMIZED:
                p.sketch_rank = 64
            m = T.SketchModel(c, path=sketch_train.DEFAULT_WEIGHTS)
            p.sketch_model = m.h.value
            _, so, _, _ = T.two_site_update_batched(c, [t(c, lo(a), T.C64) for a, _ in ab],
                                                    [t(c, lo(b), T.C64) for _, b in ab], None, p,
                                                    prev_spectra=[t(c, x, T.F64) for x in s])
            return so
        return go

    def train(c):
        g = torch.Generator().manual_seed(1)
        X, y = torch.rand((70, 35), generator=g).cuda(), torch.rand(70, generator=g).cuda() * 8
        m = T.SketchModel(c, seed=2)
        _, grad = m.grads(X, y)
        m.train_step(X, y)
        return [grad.cpu().numpy(), m.predict(X).cpu().numpy(), m.params()]

    def blocks(c):
        g = synth.rng(4, 9)
        out = []
        bl, bm = synth.u1_bond(96, 21), synth.u1_bond(80, 22)
        A = T.BsTensor.from_blocks(c, bl, bm, synth.u1_site_blocks(g, bl, bm))
        B = T.BsTensor.from_blocks(c, bm, bl, synth.u1_site_blocks(g, bm, bl))
        gate = t(c, synth.u1_gate(g), T.F64)
        p = T.update_params(chi_min=1, chi_max=96, target_trunc_err=1e-8, direction=T.DIR_LEFT, precision=T.PREC_FP32)
        for _ in range(4):        # run, recorded, replayed
            out.append(T.bs_two_site_update_batched(c, [A], [B], [gate], p)[1][0].numpy())
        return out

    def normalised(c):
        return [T.normalize_trace(c, t(c, d(n, n) + 4 * np.eye(n), T.C128)) for n in (5, 100)]

    hpd = d(40, 40)
    return {
        "contract": lambda c: [T.contract(c, t(c, d(30, 7, 500), T.C128), "abk", t(c, d(500, 11), T.C128), "kj", "jab"),
                               T.contract(c, t(c, d(4, 5, 6), T.C128), "abk", t(c, d(6, 5), T.C128), "kb", "a"),
                               T.contract(c, t(c, lo(d(30, 70)), T.C64), "ak", t(c, lo(d(70, 33)), T.C64), "kj", "ja")],
        "svd": lambda c: [T.svd(c, t(c, d(*s), T.C128), 1)[1] for s in ((30, 20), (60, 64), (20, 900))],
        "qr": lambda c: T.qr(c, t(c, d(90, 70), T.C128), 1) + T.lq(c, t(c, f(50, 80), T.F64), 1),
        "eig": lambda c: [T.eigvals(c, t(c, d(70, 70), T.C128))],
        "exp": lambda c: [T.exp(c, t(c, 0.1 * d(60, 60), T.C128), 1)],
        "inverse": lambda c: [T.inverse(c, t(c, hpd @ hpd.conj().T + np.eye(40), T.C128), 1)],
        "trace": lambda c: [T.trace(c, t(c, d(5, 6, 5), T.C128), [(0, 2)]), np.array(T.norm(c, t(c, d(300, 40), T.C128)))],
        "normalize_trace": normalised,
        "heff_fp32": matvec(T.PREC_FP32), "heff_bf16x3": matvec(T.PREC_BF16X3), "lanczos": lanczos,
        "randomized": sketch(T.SVD_RANDOMIZED), "learned": sketch(T.SVD_LEARNED), "train": train, "blocks": blocks,
    }


CALLS = ("contract", "svd", "qr", "eig", "exp", "inverse", "trace", "normalize_trace", "heff_fp32", "heff_bf16x3",
         "lanczos", "randomized", "learned", "train", "blocks")


@pytest.mark.parametrize("name", CALLS)
def test_calls_do_not_read_unwritten_workspace(T, name):
    """The same results on workspace of NaN and of zeros: the same sums in the same order, so equal up to what
    atomic additions may reorder."""
    got = []
    for byte in (0, 0xFF):
        m = Memory(T, byte)
        got.append([x if isinstance(x, np.ndarray) else x.numpy() for x in _calls(T)[name](m.refill())])
        m.ctx.close()
    for x, y in zip(*got):
        assert x.shape == y.shape and np.isfinite(y).all()
        tol = 1e-11 if x.dtype.itemsize >= (16 if x.dtype.kind == "c" else 8) else 1e-5
        assert np.abs(x - y).max() <= tol * np.abs(x).max()


# one launch of the write-back, more than one, several chunks
@pytest.mark.parametrize("n,max_batch", [(3, 0), (70, 0), (5, 2)])
def test_vidal_weights_that_are_output_spectra(T, poisoned, n, max_batch):
    """Every spectrum handle is an outer weight of two other updates of the batch and has to grow: the same results
    as with weights of their own."""
    ctx, L = poisoned.refill(), T.lib()
    a, b = draw((3, 2, 5), True, 1), draw((5, 2, 3), True, 2)
    lam = [np.sort(draw((3,), False, 10 + i) ** 2 + 0.1)[::-1].copy() for i in range(n)]
    A, B = ([T.Tensor.from_numpy(ctx, x * (1 + i), T.C128) for i in range(n)] for x in (a, b))
    wrapped = [T.Tensor.from_numpy(ctx, x, T.F64) for x in lam]
    p = T.update_params(chi_min=1, chi_max=6, direction=T.DIR_VIDAL, max_batch=max_batch)
    left, right = [(i + 1) % n for i in range(n)], [(i + 2) % n for i in range(n)]
    want = T.two_site_update_batched(ctx, A, B, None, p, lambda_left=[wrapped[i] for i in left],
                                     lambda_right=[wrapped[i] for i in right])
    P = ctypes.c_void_p * n
    own = [ctypes.c_void_p() for _ in range(n)]
    for h, w in zip(own, wrapped):
        T._check(L.tci_copy(ctx.h, w.h, ctypes.byref(h)), "tci_copy")
    Ao, Bo = ([T.Tensor.empty(ctx, T.C128, 36) for _ in range(n)] for _ in range(2))
    infos = (T.UpdateInfo * n)()
    for field, at in (("lambda_left", left), ("lambda_right", right)):
        setattr(p, field, ctypes.cast(P(*[own[i].value for i in at]), ctypes.POINTER(ctypes.c_void_p)))
    T._check(L.tci_two_site_update_batched(ctx.h, n, P(*[x.h.value for x in A]), P(*[x.h.value for x in B]), None,
                                           ctypes.byref(p), P(*[x.h.value for x in Ao]), P(*[h.value for h in own]),
                                           P(*[x.h.value for x in Bo]), infos), "tci_two_site_update_batched")
    for i in range(n):
        s = T.Tensor.empty(ctx, T.F64, 6)
        T._check(L.tci_reshape(ctx.h, own[i], 1, T._i64([infos[i].chi]), s.h), "tci_reshape")
        for x, y in ((Ao[i], want[0][i]), (s, want[1][i]), (Bo[i], want[2][i])):
            assert np.array_equal(x.numpy(), y.numpy())
        T._check(L.tci_destroy(ctx.h, own[i]), "tci_destroy")


def test_update_without_a_gate_leaves_queued_work_alone(T):
    """On a stream that does not wait for the default one: contractions whose operands are permuted in the context's
    workspace are still queued when an update without a gate of its own takes the same workspace."""
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ctx = T.Context(0, stream=side)
        x, y = (T.Tensor.from_numpy(ctx, draw((2, 1024, 1024), True, i), T.C128) for i in (1, 2))
        a, b, gate = (T.Tensor.from_numpy(ctx, z, T.C128)
                      for z in (draw((32, 2, 32), True, 3), draw((32, 2, 32), True, 4), np.eye(4) + 0j))
        out = T.Tensor.empty(ctx, T.C128, 1024 * 1024)
        p = T.update_params(chi_min=1, chi_max=32)
        want = T.contract(ctx, x, "aij", y, "alj", "il", out=out).numpy().copy()
        for _ in range(4):
            T.contract(ctx, x, "aij", y, "alj", "il", out=out)
        got = T.two_site_update_batched(ctx, [a] * 2, [b] * 2, [gate, None], p)
        assert np.array_equal(out.numpy(), want)
        for part in got[:3]:
            assert np.array_equal(part[0].numpy(), part[1].numpy())
        ctx.close()
