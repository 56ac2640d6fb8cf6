"""Edges of the kernels for small problems against numpy in 64 bits: sizes at
the tile, wave and LDS limits where each kernel's code changes."""
import numpy as np
import pytest

from paper_2512_23917_amd import synth
from gpu_util import isometry_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
U64 = 2.0 ** -53


@pytest.fixture(scope="module")
def T():
    from paper_2512_23917_amd import tci
    return tci


@pytest.fixture(scope="module")
def ctx(T):
    c = T.Context(0)
    yield c
    c.close()


def draw(shape, complex_, seed):
    g = synth.rng(31, seed)
    return synth.complex_gaussian(g, shape) if complex_ else synth.real_gaussian(g, shape)


# 32 / 33: threads per workgroup; 16 | 17 rows: lanes of a pair; 64 x 80 and 64 x 81 (complex), 64 x 224 and
# 225 (real): the largest matrices held in LDS and the smallest that are not; 1 and 2: no pair and one pair
@pytest.mark.parametrize("complex_,m,n", [(True, 1, 1), (True, 2, 5), (False, 3, 3), (True, 17, 16), (True, 31, 32),
                                          (True, 33, 33), (True, 64, 80), (True, 81, 64), (True, 300, 63),
                                          (False, 224, 64), (False, 64, 225), (False, 1000, 64), (True, 40, 5)])
def test_jacobi_svd_edges(T, ctx, complex_, m, n):
    """Each pair ends with |<a_p, a_q>| <= max(m, n) u |a_p||a_q|, so an isometry defect is at most a few of
    that; the at most 64 rotations per sweep and column leave about 1e-14 in the product of 15 sweeps."""
    a = draw((m, n), complex_, 1000 * m + n)
    u, s, vh = T.svd(ctx, T.Tensor.from_numpy(ctx, a, T.C128 if complex_ else T.F64), 1)
    u, s, vh = u.numpy(), s.numpy(), vh.numpy()
    tol = 1e-13 + 4 * max(m, n) * U64
    assert np.abs(s - np.linalg.svd(a, compute_uv=False)).max() < tol * s[0]
    assert np.linalg.norm((u * s) @ vh - a) < tol * np.linalg.norm(a)
    assert isometry_err(u) < tol and isometry_err(vh, False) < tol


# more than 64 rows: a wave per pair for up to 8 columns or from 6 rows per column on (up to 32 columns), 16 lanes
# else; 192 x 32 and 191 x 32: either side of the line; 4 and 5 x 256 rows: whole and partial batches of a lane's
# elements; 1100 x 8 and 1200 x 8 (complex): W in LDS and in global memory
@pytest.mark.parametrize("complex_,m,n", [(True, 65, 1), (True, 65, 2), (False, 70, 8), (True, 9, 80), (True, 191, 32),
                                          (True, 192, 32), (False, 97, 16), (False, 95, 16), (True, 1024, 3),
                                          (True, 1025, 7), (True, 1100, 8), (True, 1200, 8), (False, 31, 2100),
                                          (True, 33, 400), (True, 5000, 17)])
def test_jacobi_svd_long_columns(T, ctx, complex_, m, n):
    test_jacobi_svd_edges(T, ctx, complex_, m, n)


@pytest.mark.parametrize("scale", [1e-100, 1e100])
def test_jacobi_svd_far_from_one(T, ctx, scale):
    """Real matrices whose squared inner products leave the exponent range."""
    a = draw((20, 12), False, 5) * scale
    u, s, vh = T.svd(ctx, T.Tensor.from_numpy(ctx, a, T.F64), 1)
    assert np.abs(s.numpy() - np.linalg.svd(a, compute_uv=False)).max() < 1e-13 * s.numpy()[0]
    assert isometry_err(u.numpy()) < 1e-13


@pytest.mark.parametrize("complex_", [False, True])
@pytest.mark.parametrize("scale,grade", [(1e-150, 1.0), (1e-80, 1.0), (1e80, 1.0), (1e150, 1.0), (1.0, 1e-140),
                                         (1e-60, 1e-90), (1e60, 1e-130)])
@pytest.mark.parametrize("m,n", [(20, 12), (70, 33), (12, 900)])
def test_jacobi_svd_exponent_range(T, ctx, m, n, scale, grade, complex_):
    """Inner products of columns, or their squares, beyond either end of the exponent range; half of the columns
    smaller by `grade`, whose inner products are far below the others'.  As near 1, since powers of two are exact."""
    a = draw((m, n), complex_, 5) * scale
    k = min(m, n)
    np.moveaxis(a, int(m >= n), 0)[k // 2:k] *= grade
    u, s, vh = T.svd(ctx, T.Tensor.from_numpy(ctx, a, T.C128 if complex_ else T.F64), 1)
    u, s, vh = u.numpy(), s.numpy(), vh.numpy()
    tol = 1e-13 + 4 * max(m, n) * U64
    assert np.abs(s / scale - np.linalg.svd(a / scale, compute_uv=False)).max() < tol * s[0] / scale
    assert np.linalg.norm((u * (s / scale)) @ vh - a / scale) < tol * s[0] / scale * np.sqrt(k)
    assert isometry_err(u) < tol and isometry_err(vh, False) < tol


@pytest.mark.parametrize("complex_", [False, True])
@pytest.mark.parametrize("n", [3, 5, 17, 33, 63])
def test_jacobi_svd_of_a_spread_null_vector(T, ctx, n, complex_):
    """The adjacency matrix of an open chain of odd length, alone and with zero rows and columns around it: singular
    values 2 |cos(pi k / (n + 1))|, the null vector spread over (n + 1) / 2 entries of equal size."""
    chain = np.diag(np.ones(n - 1), 1) + np.diag(np.ones(n - 1), -1)
    ref = np.sort(2 * np.abs(np.cos(np.pi * np.arange(1, n + 1) / (n + 1))))[::-1]
    wide = np.zeros((n, n + 3))
    wide[:, 2:2 + n] = chain
    for a in (chain, wide, wide.T):
        code = T.C128 if complex_ else T.F64
        u, s, vh = (x.numpy() for x in T.svd(ctx, T.Tensor.from_numpy(ctx, a + 0j if complex_ else a, code), 1))
        assert np.abs(s - ref).max() < 1e-13 and np.abs((u * s) @ vh - a).max() < 1e-13
        assert isometry_err(u) < 1e-13 and isometry_err(vh, False) < 1e-13


@pytest.mark.parametrize("complex_", [False, True])
@pytest.mark.parametrize("kind", ["ones", "star", "phases", "projectors", "integers"])
@pytest.mark.parametrize("n", [4, 17, 23, 48, 64])
def test_jacobi_svd_of_exact_null_spaces(T, ctx, n, kind, complex_):
    """Matrices of low rank and exact arithmetic: the columns of the null space shrink by the unit roundoff in every
    sweep, through the smallest numbers to zero, and must leave the others as they are."""
    star = np.zeros((n, n))
    star[0, 1:] = star[1:, 0] = 1.0
    k = np.arange(n)
    half = np.ones((2, 2))
    proj = np.eye(1)
    while proj.shape[0] < n:
        proj = np.kron(proj, half)
    r = np.random.default_rng(n).integers(-2, 3, (n, max(1, n // 3)))
    a = {"ones": np.ones((n, n)), "star": star, "projectors": proj, "integers": (r @ r.T).astype(float),
         "phases": (np.diag(np.ones(n - 1), 1) + np.diag(np.ones(n - 1), -1)) * np.cos(np.outer(k, k))}[kind]
    if complex_:
        a = a * np.exp(1j * np.outer(np.arange(len(a)), np.arange(len(a)) + 1.0))
    code = T.C128 if complex_ else T.F64
    u, s, vh = (x.numpy() for x in T.svd(ctx, T.Tensor.from_numpy(ctx, a, code), 1))
    tol = 1e-13 + 4 * n * U64
    assert s.shape == (len(a),) and np.abs(s - np.linalg.svd(a, compute_uv=False)).max() < tol * s[0]
    assert np.linalg.norm((u * s) @ vh - a) < tol * np.linalg.norm(a)
    assert isometry_err(u) < tol and isometry_err(vh, False) < tol


@pytest.mark.parametrize("complex_", [False, True])
@pytest.mark.parametrize("n", [24, 32, 60])
def test_jacobi_svd_keeps_norms(T, ctx, n, complex_):
    """The rows of V^H come from about 10 n rotations each.  A rotation's c^2 + s^2 is off by 0.6 to 0.85 u rms, of
    either sign, which is 0.45 u in the norm and 0.6 u with the modulus of a complex phase: so many u times sqrt(10 n)
    rms over the rows, and a few u on average.  A phase that is short by an ulp in a third of the rotations, or a
    cosine that is long by as much, adds up to n / 2 u."""
    norms = []
    for i in range(8):
        a = draw((n, n), complex_, 100 * n + i)
        vh = T.svd(ctx, T.Tensor.from_numpy(ctx, a, T.C128 if complex_ else T.F64), 1)[2].numpy()
        norms.append(np.sqrt((np.abs(vh.astype(np.clongdouble)) ** 2).sum(axis=1)) - 1)
    assert abs(np.mean(norms)) < 6 * U64 * np.sqrt(n / 24)
    assert np.sqrt(np.mean(np.square(norms))) < (0.6 if complex_ else 0.45) * U64 * np.sqrt(10 * n)


# 64, 128, 192 (complex and real), 256 and 320 (real): row blocks held on chip; 321 .. 384 (193 .. 384 complex): first
# columns from global memory, the rest on chip; 385 and up: panels, the rest on chip
@pytest.mark.parametrize("complex_,n", [(True, n) for n in (1, 2, 3, 16, 17, 33, 64, 65, 128, 129, 192, 193, 290, 384,
                                                            385, 417)] +
                         [(False, n) for n in (1, 2, 31, 64, 65, 128, 129, 192, 193, 256, 257, 320, 321, 384, 385,
                                               500)])
def test_eigh_edges(T, ctx, complex_, n):
    """Householder reduction and its eigensolver are backward stable: eigenvalues and residuals to a small
    multiple of n u ||A||."""
    a = draw((n, n), complex_, 7 * n)
    a = (a + a.conj().T) / 2
    w, v = T.eigh(ctx, T.Tensor.from_numpy(ctx, a, T.C128 if complex_ else T.F64))
    w, v = w.numpy(), v.numpy()
    tol = (8 * n + 64) * U64 * np.linalg.norm(a, 2)
    assert np.abs(w - np.linalg.eigvalsh(a)).max() < tol
    assert np.abs(a @ v - v * w).max() < tol
    assert isometry_err(v) < (8 * n + 64) * U64


# on chip; first columns from 64 x 64 tiles, one and many of them; panels
@pytest.mark.parametrize("complex_,n", [(True, 7), (True, 192), (True, 193), (True, 200), (True, 290), (True, 384),
                                        (True, 450), (False, 320), (False, 330), (False, 384), (False, 450)])
def test_eigh_reads_the_lower_triangle(T, ctx, complex_, n):
    """Values above the diagonal that are not the conjugates of those below do not count."""
    a = draw((n, n), complex_, 9 * n)
    h = (a + a.conj().T) / 2
    given = np.tril(h) + np.triu(draw((n, n), complex_, 9 * n + 1), 1)
    code = T.C128 if complex_ else T.F64
    w, v = (x.numpy() for x in T.eigh(ctx, T.Tensor.from_numpy(ctx, given, code)))
    tol = (8 * n + 64) * U64 * np.linalg.norm(h, 2)
    assert np.abs(w - np.linalg.eigvalsh(h)).max() < tol and np.abs(h @ v - v * w).max() < tol
    assert np.abs(T.eigvalsh(ctx, T.Tensor.from_numpy(ctx, given, code)).numpy() - w).max() < tol


def check_eigh(T, ctx, a):
    n = len(a)
    w, v = (x.numpy() for x in T.eigh(ctx, T.Tensor.from_numpy(ctx, a, T.C128 if np.iscomplexobj(a) else T.F64)))
    tol = (8 * n + 64) * U64
    scale = np.linalg.norm(a, 2)
    assert np.abs(w - np.linalg.eigvalsh(a)).max() < tol * scale
    assert np.abs(a @ v - v * w).max() < tol * scale
    assert isometry_err(v) < tol


@pytest.mark.parametrize("complex_", [False, True])
@pytest.mark.parametrize("kind,n", [("ones", n) for n in (8, 25, 34, 51, 59, 192, 300, 320)] +
                         [("bipartite", n) for n in (11, 14, 17, 22, 36, 50, 65, 129, 193, 256, 330)] +
                         [("star", n) for n in (9, 64, 200)] + [("permutation", n) for n in (7, 15, 60)])
def test_eigh_of_null_spaces(T, ctx, kind, n, complex_):
    """Matrices whose reduction ends in blocks of rounding errors: eigenvectors of a null space of up to n - 1
    dimensions, and of eigenvalues that several decoupled blocks share."""
    a = np.zeros((n, n), dtype=complex if complex_ else float)
    if kind == "ones":
        a[:] = 1.0
    elif kind == "bipartite":
        a[:n // 2, n // 2:] = 1.0
        a += a.T
    elif kind == "star":
        a[0, 1:] = a[1:, 0] = 1.0
    else:
        p = np.eye(n)[np.random.default_rng(n).permutation(n)]
        a += p + p.T
    check_eigh(T, ctx, a)


@pytest.mark.parametrize("complex_", [False, True])
@pytest.mark.parametrize("kind,n", [("ring", n) for n in (4, 9, 12, 33, 100)] + [("torus", 4), ("torus", 8), ("spins", 4),
                                                                                ("spins", 6), ("spins", 8)])
def test_eigh_of_multiple_eigenvalues(T, ctx, kind, n, complex_):
    """Hopping on a ring and on a torus (pairs and quartets of equal eigenvalues) and a Heisenberg ring (multiplets)."""
    ring = np.roll(np.eye(n), 1, axis=0)
    ring = ring + ring.T
    if kind == "ring":
        a = ring
    elif kind == "torus":
        a = np.kron(ring, np.eye(n)) + np.kron(np.eye(n), ring)
    else:
        swap = np.arange(2 ** n)
        a = np.zeros((2 ** n, 2 ** n))
        for i in range(n):      # S_i . S_j = (exchange of the two spins) / 2 - 1 / 4
            j = (i + 1) % n
            bi, bj = (swap >> i) & 1, (swap >> j) & 1
            a += np.eye(2 ** n)[swap ^ ((bi ^ bj) * ((1 << i) | (1 << j)))] / 2 - np.eye(2 ** n) / 4
    check_eigh(T, ctx, a + 0j if complex_ else a)


@pytest.mark.parametrize("complex_", [False, True])
@pytest.mark.parametrize("n,seed", [(12, 0), (23, 1), (44, 2), (46, 3), (60, 4), (82, 5), (150, 6), (220, 7), (322, 8)])
def test_eigh_of_clusters_over_many_scales(T, ctx, n, seed, complex_):
    """Partial permutations with weights 1, 2, 1e-8, 1e-16 and 0, symmetrised: few distinct eigenvalues at each of the
    scales, products of the small weights among them, shared by blocks with and without small couplings."""
    g = np.random.default_rng(seed)
    for _ in range(6):
        a = np.zeros((n, n), dtype=complex if complex_ else float)
        a[np.arange(n), g.permutation(n)] = g.choice([1.0, -1.0, 2.0, 1e-8, 1e-16, 0.0], n)
        if complex_:
            a *= np.exp(1j * (np.arange(n)[:, None] - np.arange(n)))
        check_eigh(T, ctx, (a + a.conj().T) / 2)


@pytest.mark.parametrize("n,scale", [(9, 1.0), (40, 1e-120), (40, 1e120), (130, 1.0)])
def test_eigvalsh_of_diagonals(T, ctx, n, scale):
    """Diagonal matrices with values over 200 decades, both signs, repeated values and zeros: the reduction
    leaves them as they are, and bisection resolves every value to a few ulps of itself."""
    d = 10.0 ** -np.linspace(0, 100, n) * np.where(np.arange(n) % 3 == 1, -1.0, 1.0) * scale
    d[n // 2:n // 2 + 2] = 0.0
    d[-1] = d[0]
    w = T.eigvalsh(ctx, T.Tensor.from_numpy(ctx, np.diag(d), T.F64)).numpy()
    ref = np.sort(d)
    assert np.all(np.abs(w - ref) <= 8 * U64 * np.abs(ref))


# L lanes per eigenvalue: 64 up to 1024 eigenvalues, 16 up to 8192, 4 up to 32768, 1 above
@pytest.mark.parametrize("batch,chi", [(2, 40), (60, 40), (64, 130), (64, 300)])
def test_singular_values_of_padded_batches(T, ctx, batch, chi):
    """Two-site updates of tensors whose last bond indices are zero: exact zero eigenvalues beside a graded
    spectrum, for every number of lanes per eigenvalue.  The Gram route leaves n u of the largest square."""
    n = 2 * chi
    p = T.update_params(chi_min=1, chi_max=n, target_trunc_err=0.0, direction=T.DIR_LEFT, precision=T.PREC_FP64)
    A, B, ref = [], [], []
    for i in range(2):
        a, b = draw((chi, 2, chi), False, 50 + i), draw((chi, 2, chi), False, 90 + i)
        a[chi - 9:] = 0.0
        b *= 10.0 ** -np.linspace(0, 4, chi)[:, None, None]
        ref.append(np.linalg.svd(a.reshape(n, chi) @ b.reshape(chi, n), compute_uv=False))
        A.append(T.Tensor.from_numpy(ctx, a, T.F64))
        B.append(T.Tensor.from_numpy(ctx, b, T.F64))
    A, B, ref = (x * (batch // 2) for x in (A, B, ref))
    _, s, _, info = T.two_site_update_batched(ctx, A, B, None, p)
    for x, r, f in zip(s, ref, info):
        x = x.numpy() * np.sqrt(f.norm2)
        k = chi - 20    # well above the rounding level of the Gram matrix
        assert np.abs(x[:k] ** 2 - r[:k] ** 2).max() < 8 * n * U64 * r[0] ** 2
        assert np.all(x[chi:] ** 2 < 8 * n * U64 * r[0] ** 2)


# complex FP64 tiles are 128 x 64, 64 x 64 or 32 x 32 by the size of the launch: remainders of each tile, a long inner
# dimension (split) on a small output, and sizes that choose each shape; the four with K <= 32 and at most 2^17
# multiply-adds take the one-launch path
@pytest.mark.parametrize("complex_,m,n,k", [(True, 1, 1, 1), (True, 33, 31, 17), (True, 31, 65, 1), (True, 129, 63, 300),
                                            (True, 520, 530, 40), (True, 1100, 1000, 33), (True, 2050, 2047, 19),
                                            (False, 33, 70, 5), (False, 65, 64, 1000), (False, 1030, 1040, 20),
                                            (False, 2300, 2200, 18), (True, 40, 40, 3000)])
def test_fp64_product_tiles(T, ctx, complex_, m, n, k):
    """Sums of k products: error at most about 2 k u of sum |a||b| per element (four real products when complex)."""
    a, b = draw((m, k), complex_, m + k), draw((k, n), complex_, n + 2 * k)
    dt = T.C128 if complex_ else T.F64
    c = T.contract(ctx, T.Tensor.from_numpy(ctx, a, dt), "ik", T.Tensor.from_numpy(ctx, b, dt), "kj", "ij").numpy()
    assert np.all(np.abs(c - a @ b) <= 4 * (k + 2) * U64 * (np.abs(a) @ np.abs(b)))


# the same kernel below one tile: a single element, inner dimensions shorter than a k tile, remainders of the 32 x 32
# tile; the result shares memory with an operand, which keeps such small products off the one-launch path
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (7, 5, 3), (33, 31, 17), (31, 65, 1), (33, 70, 5), (16, 16, 15),
                                   (32, 32, 16), (64, 33, 31), (1, 200, 2)])
@pytest.mark.parametrize("complex_", [True, False])
def test_fp64_products_below_one_tile(T, ctx, m, n, k, complex_):
    a, b = draw((m, k), complex_, m + k), draw((k, n), complex_, n + 2 * k)
    dt = T.C128 if complex_ else T.F64
    buf = torch.zeros(m * max(n, k), dtype=T.TORCH_OF[dt], device="cuda")
    buf[:m * k] = torch.from_numpy(a.reshape(-1))
    ta, out = T.Tensor(ctx, buf[:m * k].view(m, k)), T.Tensor(ctx, buf)
    c = T.contract(ctx, ta, "ik", T.Tensor.from_numpy(ctx, b, dt), "kj", "ij", out=out).numpy()
    assert np.all(np.abs(c - a @ b) <= 4 * (k + 2) * U64 * (np.abs(a) @ np.abs(b)))


def test_profiled_work_of_a_lower_triangle(T, ctx):
    """A complex Gram matrix of order 128 runs in 32 x 32 tiles, without those whose columns are 64 or more beyond
    their rows: one tile of the first tile row is left out."""
    a = draw((128, 128), True, 3)
    T.profile_enable(ctx, True)
    try:
        T.trunc_svd(ctx, T.Tensor.from_numpy(ctx, a, T.C128), 1, 1, 20)
        count, _, work = T.profile_query(ctx, "svd_gram:c128_fp64")
    finally:
        T.profile_enable(ctx, False)
    assert count == 1 and work == 8 * 128 * (128 * 128 - 32 * 32)


# 64 samples per stage, one sample per workgroup up to 512 and four above; several stages
@pytest.mark.parametrize("n", [1, 63, 65, 512, 513, 2051])
def test_sketch_gradients(T, ctx, n):
    """FP32 sums of n products of values of order one: error at most about n 2^-24 of the sum of magnitudes, which
    a gradient of the mean bounds by 2^-24 n times its largest entries; a few thousand ulps here."""
    g = torch.Generator().manual_seed(n)
    X, t = torch.rand((n, 35), generator=g) * 2 - 1, torch.rand(n, generator=g) * 8
    m = T.SketchModel(ctx, seed=3)
    flat = torch.from_numpy(m.params()).double().requires_grad_(True)
    h, at = X.double(), 0
    for k, (r, c) in enumerate(((128, 35), (128, 128), (1, 128))):
        h = h @ flat[at:at + r * c].reshape(r, c).t() + flat[at + r * c:at + r * c + r]
        h = torch.nn.functional.gelu(h) if k < 2 else h
        at += r * c + r
    u = t.double() - h[:, 0]
    ref = torch.maximum(0.9 * u, -0.1 * u).mean()
    ref.backward()
    loss, grad = m.grads(X, t)
    ref = float(ref.detach())
    assert abs(loss - ref) < 2e-5 * ref
    err = (grad.cpu().double() - flat.grad).abs().max() / flat.grad.abs().max()
    assert float(err) < 2e-5
    assert float((m.predict(X).cpu().double() - h[:, 0].detach()).abs().max()) < 2e-5 * float(h.detach().abs().max())


# one launch up to 32 summed terms, 64 with permuted operands, 2^17 multiply-adds; the general path above
@pytest.mark.parametrize("la,lb,lc,dims", [
    ("ab", "ab", "", dict(a=4, b=16)), ("ab", "bc", "ac", dict(a=1, b=1, c=1)), ("ab", "bc", "ca", dict(a=5, b=33, c=7)),
    ("sabc", "bx", "saxc", dict(s=2, a=3, b=16, c=4, x=16)), ("cabs", "cds", "dab", dict(a=3, b=2, c=4, d=9, s=16)),
    ("cabs", "cds", "dab", dict(a=3, b=2, c=4, d=9, s=17)), ("a", "b", "ba", dict(a=300, b=437)),
    ("abc", "cbd", "da", dict(a=64, b=8, c=8, d=32)), ("abc", "cbd", "da", dict(a=64, b=8, c=8, d=33)),
    ("ab", "bc", "ac", dict(a=64, b=32, c=64)), ("ab", "bc", "ac", dict(a=64, b=33, c=64)),
    ("abcd", "efgh", "hagbfced", dict.fromkeys("abcdefgh", 2))])
@pytest.mark.parametrize("complex_", [True, False])
def test_small_contractions(T, ctx, la, lb, lc, dims, complex_):
    a, b = (draw([dims[x] for x in lab], complex_, 11 + i) for i, lab in enumerate((la, lb)))
    dt = T.C128 if complex_ else T.F64
    ta, tb = T.Tensor.from_numpy(ctx, a, dt), T.Tensor.from_numpy(ctx, b, dt)
    ref, mag = (np.einsum(f"{la},{lb}->{lc}", x, y) for x, y in ((a, b), (np.abs(a), np.abs(b))))
    k = max(1, int(np.prod([dims[x] for x in set(la) & set(lb)])))
    c = T.contract(ctx, ta, la, tb, lb, lc).numpy()
    assert c.shape == ref.shape and np.all(np.abs(c - ref) <= 4 * (k + 2) * U64 * mag)


def test_small_contraction_into_shared_memory(T, ctx):
    """The result over an operand's handle, and over its memory through another wrapped tensor."""
    a, b = draw((4, 6), True, 1), draw((6, 6), True, 2)
    ref = np.einsum("ab,bc->ca", a, b)
    ta, tb = T.Tensor.from_numpy(ctx, a, T.C128), T.Tensor.from_numpy(ctx, b, T.C128)
    buf = ta.buf
    shared = T.Tensor(ctx, buf.view(-1), shape=[24])
    assert np.abs(T.contract(ctx, ta, "ab", tb, "bc", "ca", out=shared).numpy() - ref).max() < 1e-13
    ta = T.Tensor.from_numpy(ctx, a, T.C128)
    assert np.abs(T.contract(ctx, ta, "ab", tb, "bc", "ca", out=ta).numpy() - ref).max() < 1e-13


# one block up to order 64, two launches above
@pytest.mark.parametrize("n", [1, 3, 64, 65, 300])
@pytest.mark.parametrize("dt", ["F32", "F64", "C64", "C128"])
def test_normalize_trace(T, ctx, n, dt):
    a = draw((n, n), dt.startswith("C"), n) + np.eye(n) * 4
    a = a.astype(T.NUMPY_OF[getattr(T, dt)])
    t = T.normalize_trace(ctx, T.Tensor.from_numpy(ctx, a, getattr(T, dt)))
    ref = a.astype(np.complex128) / np.trace(a.astype(np.complex128))
    u = 2.0 ** -24 if dt in ("F32", "C64") else U64
    assert np.abs(t.numpy() - ref).max() <= (n + 8) * U64 * np.abs(ref).max() * np.sqrt(n) + 2 * u * np.abs(ref).max()
    with pytest.raises(T.TciError):
        T.normalize_trace(ctx, T.Tensor.from_numpy(ctx, np.zeros((2, 3)), T.F64))


@pytest.mark.parametrize("n", [3, 100])
@pytest.mark.parametrize("scale", [1e-300, 1e-160, 1e160, 1e300, 1e-200j, -1e200j, 1e180 * (1 - 1e-9j)])
def test_normalize_trace_far_from_one(T, ctx, n, scale):
    """Traces whose squared modulus leaves the exponent range, real and imaginary parts of either size."""
    a = draw((n, n), True, n) + np.eye(n) * 4
    t = T.normalize_trace(ctx, T.Tensor.from_numpy(ctx, a * scale, T.C128))
    ref = a / np.trace(a)
    # the trace to about n u of the sum of moduli, four roundings of the division, the product and the scaling
    assert np.abs(t.numpy() - ref).max() <= (n + 16) * U64 * np.abs(ref).max() * np.sqrt(n)


# 64 tensors per launch; complex64 factors with an odd element count (8-byte copies); an update without a gate
@pytest.mark.parametrize("batch,dt", [(1, "C64"), (63, "F32"), (65, "C64"), (130, "F64")])
def test_update_batches_beyond_one_table(T, ctx, batch, dt):
    """Every update of a batch equals the same update alone, up to the rounding of a single-precision result."""
    code = getattr(T, dt)
    prec = T.PREC_FP64 if dt == "F64" else T.PREC_FP32
    p = T.update_params(chi_min=1, chi_max=4, direction=T.DIR_LEFT, precision=prec, max_batch=128)
    up = lambda x: T.Tensor.from_numpy(ctx, x.astype(T.NUMPY_OF[code]), code)  # noqa: E731
    c = dt.startswith("C")
    A = [up(draw((3, 2, 5), c, 3 * i)) for i in range(batch)]
    B = [up(draw((5, 2, 3), c, 3 * i + 1)) for i in range(batch)]
    G = [up(draw((2, 2, 2, 2), c, 3 * i + 2)) if i % 3 else None for i in range(batch)]
    Ao, so, Bo, info = T.two_site_update_batched(ctx, A, B, G, p)
    tol = 1e-12 if dt == "F64" else 2e-6
    for i in range(batch):
        a1, s1, b1, _ = T.two_site_update_batched(ctx, [A[i]], [B[i]], [G[i]], p)
        assert Ao[i].numpy().shape == (3, 2, 4) and info[i].chi == 4
        for x, y in ((Ao[i], a1[0]), (so[i], s1[0]), (Bo[i], b1[0])):
            assert np.abs(x.numpy() - y.numpy()).max() <= tol


# left / right products of the split-BF16x3 planes: 1 x 1, 8 x 3 and 33 x 70 in 32 x 32 tiles, 250 x 200 in
# 64 x 64 and 32 x 32, 400 x 390 in 128 x 128 and 64 x 64; bonds that leave a remainder in every tile
@pytest.mark.parametrize("complex_", [True, False])
@pytest.mark.parametrize("cl,cr", [(1, 1), (8, 3), (33, 70), (250, 200), (400, 390)])
def test_plane_product_tiles(T, ctx, cl, cr, complex_):
    """With 8-bit significands the split leaves 2^-18 of each factor and drops a product of at most 2^-18: 3 x 2^-18
    per term and step, 3.5e-5 in three steps, of random sign; single-precision sums add far less.  Bounded by the
    sum of the terms' moduli for each element, and by the norm where there are enough of them to average."""
    from oracle import dmrg as odmrg
    lo, code = (np.complex64, T.C64) if complex_ else (np.float32, T.F32)
    w = synth.heisenberg_mpo()
    arrs = [draw((cl, 5, cl), complex_, cl), w if complex_ else w.real, draw((cr, 5, cr), complex_, cr + 1),
            draw((cl, 2, 2, cr), complex_, cl + 2)]
    left, w, right, x = (np.asarray(a).astype(lo) for a in arrs)
    l64, w64, r64, x64 = (a.astype(np.complex128) for a in (left, w, right, x))
    ref = odmrg.heff_apply(l64, w64, w64, r64, x64)
    up = lambda a: T.Tensor.from_numpy(ctx, a, code)  # noqa: E731
    ctx.set_precision(T.PREC_BF16X3)
    try:
        y = T.heff_matvec(ctx, up(left), up(w), up(w), up(right), up(x)).numpy()
    finally:
        ctx.set_precision(T.PREC_FP32)
    err = np.abs(y - ref)
    terms = odmrg.heff_apply(*(np.abs(a) for a in (l64, w64, w64, r64, x64))).real
    assert (err <= 2 * 3.5e-5 * terms + 1e-30).all()
    if cl > 1:
        assert np.linalg.norm(err) <= 3.5e-5 * np.linalg.norm(ref)
        assert err.max() <= 40 * 3.5e-5 * np.linalg.norm(ref) / np.sqrt(ref.size)
