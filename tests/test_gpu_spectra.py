"""Multi-mode SVD invariants and tensor matching (Section 4.2) on the GPU,
through the C ABI, against the oracle.

Spectra: every eigenvalue sigma^2 within 1e-9 of the unfolding's largest
(the fp64 Gram sums at most a few million fp32 products, each exact, and the
tridiagonal reduction and bisection are backward stable, so the error is far
below that).  Matching: the GPU's decisions equal the oracle's on the same
spectra, and planted permutations match while perturbed tensors do not.
"""
import ctypes
import itertools

import numpy as np
import pytest

from gpu_util import log
from oracle import spectra as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2512_08365_amd as mag
    mag.version()
    yield


def _gpu_lists(arrays):
    import torch
    import paper_2512_08365_amd as mag
    ts = [torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda() for a in arrays]
    spec, lay = mag.invariants(ts)
    flat = spec.cpu().numpy()
    out, o = [], 0
    for lens in lay:
        lst = []
        for n in lens:
            lst.append(flat[o:o + n])
            o += n
        out.append(lst)
    assert o == flat.size
    return ts, spec, out


def _assert_spectra(got, want, label):
    assert len(got) == len(want), label
    for g, w in zip(got, want):
        assert g.shape == w.shape, label
        top = max(float(w[0]), 1e-300) ** 2
        err = np.abs(g.astype(np.float64) ** 2 - w ** 2).max()
        assert err <= 1e-9 * top, (label, err / top)
        assert np.all(np.diff(g) <= 0), label  # descending


SHAPES = [(5,), (1, 1), (3, 7), (16, 16), (17, 33), (2, 3, 4), (4, 1, 9), (8, 64, 128),
          (3, 5, 2, 7), (2, 3, 2, 3, 2), (1, 4, 1, 5, 1), (100, 600), (511, 40), (512, 512),
          (2, 256, 4096), (20, 25, 700),
          # Gram sides in (64, 128], each made by one workgroup per column
          # chunk: just above 64, ragged column chunks and steps, rows from two
          # modes, both gather directions of the attention-shaped tensors
          (65, 3000), (3, 40, 1100), (128, 2049), (32, 128, 128),
          # Gram sides above 512: the many-workgroup reduction (one or two large
          # unfoldings beside a small one, a side not a multiple of the blocks)
          (600, 700), (2, 600, 700), (1030, 1100)]


@pytest.mark.parametrize("shape", SHAPES)
def test_spectra_match_the_oracle(shape):
    rng = np.random.default_rng(sum(shape))
    T = rng.standard_normal(shape).astype(np.float32)
    if len(shape) >= 2:
        T[..., 0] *= 50.0  # a spread of singular values
    log(f"[spectra] shape {shape}")
    _, _, (got,) = _gpu_lists([T])
    _assert_spectra(got, S.invariants(T), f"{shape}")


def test_closed_forms_on_the_gpu():
    rng = np.random.default_rng(4)
    vs = [rng.standard_normal(n).astype(np.float32) for n in (6, 9, 5)]
    R1 = np.einsum("i,j,k->ijk", *vs)
    H = np.array([[1, 1, 1, 1], [1, -1, 1, -1], [1, 1, -1, -1], [1, -1, -1, 1]], np.float32) / 2
    _, _, (r1, h) = _gpu_lists([R1, H.reshape(2, 2, 2, 2)])
    norm = float(np.prod([np.linalg.norm(v.astype(np.float64)) for v in vs]))
    for s in r1:
        assert abs(s[0] - norm) <= 1e-6 * norm and np.all(s[1:] <= 1e-6 * norm)
    assert np.allclose(h[S.canonical_masks(4).index(0b0011)], 1.0, atol=1e-7)


@pytest.mark.parametrize("k,l", [(128, 600), (96, 257)])
def test_clustered_spectra_whole_triangle_sides(k, l):
    """Gram sides in (64, 128] (one workgroup per column chunk makes the whole
    triangle) with repeated and clustered singular values, where bisection
    has to separate equal eigenvalues: against the oracle on the same fp32
    data, and against the singular values the matrix was built from (its
    fp32 rounding moves them by about 1e-7 relative)."""
    rng = np.random.default_rng(k + l)
    q = rng.standard_normal((k, k))
    u, _ = np.linalg.qr(q)
    w, _ = np.linalg.qr(rng.standard_normal((l, k)))
    parts = [np.full(k // 6, 10.0), np.full(k // 4, 5.0), 1.0 + 1e-6 * np.arange(k // 6),
             np.linspace(1.5, 3.0, k // 6)]
    sv = np.concatenate(parts)
    sv = np.concatenate([sv, np.full(k - sv.size, 1e-3)])
    X = ((u * sv) @ w.T).astype(np.float32)
    log(f"[spectra] clustered {k} x {l}")
    _, _, (got,) = _gpu_lists([X])
    _assert_spectra(got, S.invariants(X), f"clustered {k} x {l}")
    want = np.sort(sv)[::-1]
    assert np.abs(got[0].astype(np.float64) - want).max() <= 1e-5 * want[0]


def test_mixed_batch_in_one_call():
    """One call over tensors of every Gram class (one 32-side block, the whole
    triangle for sides in (64, 128], 64-side blocks, and sides above 512 on
    the many-workgroup path), so the library's reordering of the unfoldings
    by class and its numbering of the eigenvalue work items (large sides have
    none) are checked against each tensor's own oracle lists, in input order."""
    rng = np.random.default_rng(21)
    shapes = [(5,), (100, 600), (600, 700), (3, 40, 1100), (17, 33), (2, 256, 4096), (65, 80),
              (8, 64, 128), (1, 1)]
    Ts = [rng.standard_normal(sh).astype(np.float32) for sh in shapes]
    log(f"[spectra] mixed batch {shapes}")
    _, _, got = _gpu_lists(Ts)
    assert len(got) == len(Ts)
    for T, g, sh in zip(Ts, got, shapes):
        _assert_spectra(g, S.invariants(T), f"mixed {sh}")


def test_matching_planted_permutations():
    rng = np.random.default_rng(11)
    A = [rng.standard_normal(s).astype(np.float32) for s in
         [(4, 6, 5), (3, 3, 8), (2, 5, 2, 3), (30, 20), (6, 8, 10)]]
    B = []
    truth = np.zeros((len(A), 0), bool)
    cols = []
    for i, a in enumerate(A):
        perm = tuple(rng.permutation(a.ndim))
        B.append(np.ascontiguousarray(np.transpose(a, perm)))  # a layout change: matches
        cols.append(i)
        bad = a.copy()
        bad.flat[7] += 1e-2 * np.abs(a).max()  # a different tensor: does not
        B.append(bad)
        cols.append(-1)
    B.append(A[0].reshape(6, 4, 5).copy())  # regrouped modes: not a layout change
    cols.append(-1)
    import paper_2512_08365_amd as mag
    ta, sa, la = _gpu_lists(A)
    tb, sb, lb = _gpu_lists(B)
    got = mag.match(ta, sa, tb, sb, 1e-5).cpu().numpy()
    want = np.array([[S.match(x, y, 1e-5) for y in lb] for x in la], np.uint8)
    assert np.array_equal(got, want)  # the same decisions on the same spectra
    planted = np.array([[c == i for c in cols] for i in range(len(A))], np.uint8)
    assert np.array_equal(got, planted), (got, planted)


@pytest.mark.parametrize("shape", [(3, 4, 5, 2)])
def test_every_permutation_matches_on_the_gpu(shape):
    import paper_2512_08365_amd as mag
    rng = np.random.default_rng(5)
    T = rng.standard_normal(shape).astype(np.float32)
    perms = [np.ascontiguousarray(np.transpose(T, p)) for p in itertools.permutations(range(4))]
    ta, sa, _ = _gpu_lists([T])
    tb, sb, _ = _gpu_lists(perms)
    assert mag.match(ta, sa, tb, sb, 1e-5).cpu().numpy().all()


def test_unsupported_shapes_are_rejected():
    import torch
    import paper_2512_08365_amd as mag
    with pytest.raises(mag.MagnetonError) as e:
        # min(M, N) = 8193 > MAG_SVD_MAX_K (refused before any device work)
        mag.invariants([torch.empty((8193, 8194), device="cuda")])
    assert e.value.code == -2
    with pytest.raises(mag.MagnetonError):
        mag.invariants([torch.zeros((2,) * 6, device="cuda")])  # rank 6


def test_large_rank_deficient_unfolding():
    """A Gram side above 512 whose matrix is rank-deficient (zero rows, and
    rows repeated): Householder steps whose column is already reduced are
    skipped, and the zero eigenvalues come out within the bound."""
    rng = np.random.default_rng(12)
    T = np.zeros((700, 800), np.float32)
    T[:300] = rng.standard_normal((300, 800)).astype(np.float32)
    T[300:350] = T[:50]  # repeated rows
    T[:, :3] *= 40.0
    log("[spectra] rank-deficient 700 x 800")
    _, _, (got,) = _gpu_lists([T])
    _assert_spectra(got, S.invariants(T), "rank-deficient 700 x 800")


# Sides of the one-workgroup classes in registers (32, 64, 128, 192) and their
# edges, and the smallest matrices
@pytest.mark.parametrize("K", [1, 2, 3, 4, 31, 32, 33, 63, 64, 65, 127, 128, 129, 160, 191, 192])
def test_register_reduced_sides(K):
    rng = np.random.default_rng(K)
    T = rng.standard_normal((K, K + 11)).astype(np.float32)
    T[K // 2] *= 1e-3
    if K > 8:
        T[3] = T[1]  # a rank deficiency
    log(f"[spectra] register-reduced side {K}")
    _, _, (got,) = _gpu_lists([T])
    _assert_spectra(got, S.invariants(T), f"side {K}")


# Sides of the group reduction's classes and their edges: the smallest, one member
# with one row more than the others (257), members without their last rows (489,
# 505, 1017), whole classes, and one past each (reduced in two classes, one taking
# over from the other); above 2048 some rows are in LDS, above 3072 in memory too
@pytest.mark.parametrize("K", [193, 194, 257, 489, 505, 512, 513, 1017, 1024, 1025, 2048, 2049])
def test_group_reduced_sides(K):
    rng = np.random.default_rng(K)
    T = rng.standard_normal((K, K + 37)).astype(np.float32)
    T[:, :5] *= 30.0
    T[3] *= 1e-3
    log(f"[spectra] group-reduced side {K}")
    _, _, (got,) = _gpu_lists([T])
    _assert_spectra(got, S.invariants(T), f"side {K}")


# the largest class, and a side beyond it (device-wide steps down to 4096, then
# the group): eigenvalues of the fp64 Gram matrix, within a few thousand
# rounding units of the largest (a sum of 4,200 products, then the reduction)
@pytest.mark.parametrize("K", [3072, 3073, 4096, 4099])
def test_group_reduced_large_sides(K):
    rng = np.random.default_rng(K)
    T = rng.standard_normal((K, K + 100)).astype(np.float32)
    log(f"[spectra] group-reduced side {K}")
    _, _, (got,) = _gpu_lists([T])
    X = T.astype(np.float64)
    want = np.linalg.eigvalsh(X @ X.T)[::-1]
    lam = np.asarray(got[0]) ** 2
    assert np.max(np.abs(lam - want)) <= 1e-12 * want[0]


def test_group_reduction_batch():
    """More groups than fit at once, of several classes, beside sides that one
    workgroup reduces: launch rounds and the hand-over between classes."""
    rng = np.random.default_rng(31)
    shapes = [(300, 310)] * 9 + [(700, 720), (130, 140), (520, 530), (60, 400), (1100, 1120),
                                 (512, 700), (2, 200, 3, 150)]
    Ts = [rng.standard_normal(sh).astype(np.float32) for sh in shapes]
    log(f"[spectra] group batch {shapes}")
    _, _, got = _gpu_lists(Ts)
    for T, g, sh in zip(Ts, got, shapes):
        _assert_spectra(g, S.invariants(T), f"group batch {sh}")


def test_zero_and_diagonal_tensors():
    """Splitting tridiagonal forms: all zeros, a diagonal matrix, and repeated
    diagonal entries (every off-diagonal entry zero)."""
    Z = np.zeros((200, 210), np.float32)
    D = np.zeros((150, 160), np.float32)
    D[np.arange(150), np.arange(150)] = np.linspace(1.0, 2.0, 150).astype(np.float32)
    R = np.zeros((40, 50), np.float32)
    R[np.arange(40), np.arange(40)] = np.repeat(np.float32([1.0, 0.0, 3.0, 1e-3]), 10)
    _, _, (z, d, r) = _gpu_lists([Z, D, R])
    assert np.all(np.asarray(z[0]) == 0.0)
    _assert_spectra(d, S.invariants(D), "diagonal")
    _assert_spectra(r, S.invariants(R), "repeated diagonal")


@pytest.mark.parametrize("K", [6, 40, 150, 300, 600, 1100])
def test_small_values_of_diagonal_tensors(K):
    """Values from 1 down to 1e-18 and zeros on the diagonal, in any order: the
    Gram matrix is diagonal and exact (squares of fp32 values), so that every
    value is its square's root to a few units of rounding, and zero is zero."""
    rng = np.random.default_rng(K)
    v = np.zeros(K, np.float32)
    v[:K // 2] = np.logspace(0, -18, K // 2)
    v = rng.permutation(v)
    D = np.zeros((K, K + 8), np.float32)
    D[np.arange(K), np.arange(K)] = v
    log(f"[spectra] diagonal, small values, side {K}")
    _, _, (got,) = _gpu_lists([D])
    want = np.sort(v.astype(np.float64))[::-1]
    assert np.all(got[0][want == 0] == 0.0)
    nz = want > 0
    # (half of the eigenvalue's two units, and the root's own)
    assert np.abs(got[0][nz] / want[nz] - 1.0).max() <= 4 * np.finfo(float).eps


@pytest.mark.parametrize("n1,n2", [(20, 15), (100, 50), (200, 120), (300, 330)])
def test_small_block_of_a_block_tensor(n1, n2):
    """Two blocks that share no row or column, the second 1e-12 of the first, and
    rows of zeros: each block's values are as near as those of the block by
    itself would be, and the zero rows' are zero."""
    rng = np.random.default_rng(n1)
    b1 = rng.standard_normal((n1, n1 + 3)).astype(np.float32)
    b2 = (1e-12 * rng.standard_normal((n2, n2 + 5))).astype(np.float32)
    T = np.zeros((n1 + n2 + 4, n1 + n2 + 9), np.float32)
    T[:n1, :n1 + 3] = b1
    T[n1:n1 + n2, n1 + 3:n1 + n2 + 8] = b2
    log(f"[spectra] blocks of sides {n1} and {n2}")
    _, _, (got,) = _gpu_lists([T])
    for lo, b in ((0, b1), (n1, b2)):
        X = b.astype(np.float64)
        want = np.linalg.eigvalsh(X @ X.T)[::-1]
        lam = got[0][lo:lo + len(b)] ** 2
        assert np.abs(lam - want).max() <= 1e-12 * want[0]
    assert np.all(got[0][n1 + n2:] == 0.0)


def test_one_workgroup_each_in_a_large_batch():
    """Many sides in (192, 512]: one workgroup each, from memory, where groups would
    take several launches after one another."""
    rng = np.random.default_rng(64)
    Ts = [rng.standard_normal((200 + i % 3, 215)).astype(np.float32) for i in range(64)]
    log("[spectra] 64 sides of 200 to 202")
    _, _, got = _gpu_lists(Ts)
    for i, (T, g) in enumerate(zip(Ts, got)):
        _assert_spectra(g, S.invariants(T), f"large batch {i}")


@pytest.mark.parametrize("n", [3, 300, 700, 1030])
def test_device_wide_reduction_alone(n):
    """The device-wide steps all the way (where no group can run: a masked stream,
    a refused launch): the tridiagonal form has the matrix's eigenvalues."""
    import torch
    from paper_2512_08365_amd import _native
    launch = getattr(_native.load(), "_ZN3mag16launch_svd_largeEPdiiS0_S0_S0_P12ihipStream_t")
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, n))
    A = torch.from_numpy(X + X.T).cuda()
    want = np.linalg.eigvalsh(X + X.T)
    d, e2 = (torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(2))
    scratch = torch.zeros((2 + (n + 255) // 256) * n + 8, dtype=torch.float64, device="cuda")
    log(f"[spectra] device-wide reduction of side {n}")
    rc = launch(ctypes.c_void_p(A.data_ptr()), n, n - 2, ctypes.c_void_p(scratch.data_ptr()),
                ctypes.c_void_p(d.data_ptr()), ctypes.c_void_p(e2.data_ptr()),
                ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    off = np.sqrt(e2.cpu().numpy()[:-1])
    T = np.diag(d.cpu().numpy()) + np.diag(off, 1) + np.diag(off, -1)
    assert np.abs(np.linalg.eigvalsh(T) - want).max() <= 1e-12 * np.abs(want).max()


class _TriMatrix(ctypes.Structure):
    _fields_ = [("A", ctypes.c_void_p), ("d", ctypes.c_void_p), ("e2", ctypes.c_void_p),
                ("words", ctypes.c_void_p), ("lda", ctypes.c_int64), ("n", ctypes.c_int32),
                ("tag", ctypes.c_uint32)]


@pytest.mark.parametrize("sides,lost_at", [((600,), 0), ((600, 300), 40), ((1100, 700), 75),
                                           ((300,), -1)])
def test_members_that_lose_touch_leave(sides, lost_at):
    """One member of every group leaves at a step, as if it had waited too long:
    the others follow within about a second, the launch that would have taken over does
    at once, and the call is marked.  Never lost: the tridiagonal form has the
    matrix's eigenvalues."""
    import time

    import torch
    from paper_2512_08365_amd import _native
    launch = getattr(_native.load(),
                     "_ZN3mag17launch_tri_groupsEPNS_9TriMatrixEiiPiP12ihipStream_t")
    rng = np.random.default_rng(lost_at + 2)
    log(f"[spectra] groups {sides} lose a member at step {lost_at}")
    keep, m = [], (_TriMatrix * len(sides))()
    for t, n in zip(m, sides):
        X = rng.standard_normal((n, n))
        A = torch.from_numpy(X + X.T).cuda()
        d, e2 = (torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(2))
        words = torch.zeros(8 * (4096 + 128), dtype=torch.int64, device="cuda")
        keep.append((A.clone(), A, d, e2, words))
        t.A, t.d, t.e2, t.words = A.data_ptr(), d.data_ptr(), e2.data_ptr(), words.data_ptr()
        t.lda, t.n, t.tag = n, n, 0
    failed = torch.zeros(1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    rc = launch(m, len(sides), lost_at, ctypes.c_void_p(failed.data_ptr()),
                ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert rc == 0 and time.perf_counter() - t0 < 1.8
    assert bool(failed.item()) == (lost_at >= 0)
    if lost_at < 0:
        for A0, _, d, e2, _ in keep:
            off = e2[:-1].sqrt()
            T = torch.diag(d) + torch.diag(off, 1) + torch.diag(off, -1)
            got, want = torch.linalg.eigvalsh(T.cpu()), torch.linalg.eigvalsh(A0.cpu())
            assert float((got - want).abs().max()) <= 1e-12 * float(want.abs().max())
    # the next call is as any other
    T = rng.standard_normal((300, 320)).astype(np.float32)
    _, _, (got,) = _gpu_lists([T])
    _assert_spectra(got, S.invariants(T), "after")


def test_invariants_of_two_threads():
    """Two host threads, each with a stream of its own, whose groups fill the
    device by themselves: every call's spectra are its own."""
    import threading

    import torch
    import paper_2512_08365_amd as mag
    rng = np.random.default_rng(17)
    sets = [[rng.standard_normal((512, 530)).astype(np.float32) for _ in range(8)] +
            [rng.standard_normal((20, 1000)).astype(np.float32)],
            [rng.standard_normal((1500, 1600)).astype(np.float32), np.eye(40, 50, dtype=np.float32)]]
    dev = [[torch.from_numpy(x).cuda() for x in s] for s in sets]
    want = [mag.invariants(ts)[0].cpu().numpy() for ts in dev]
    got = [[], []]
    log("[spectra] two threads")

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(4):
                got[i].append(mag.invariants(dev[i])[0].cpu().numpy())

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(2):
        assert len(got[i]) == 4
        for g in got[i]:  # (the order in which a Gram matrix's chunks are added differs)
            np.testing.assert_allclose(g ** 2, want[i] ** 2, rtol=0, atol=1e-12 * want[i].max() ** 2)
