"""The direct spectral solver (binary32, default schedule): eigenvalues by
sections and secants of the determinant, eigenvectors by twisted
factorizations, against the binary64 oracle -- at the edges of its blocks of
eight rows and of the team shapes, on split and degenerate spectra that it
hands to the divide step, and at eigenvalue distances around that line."""
import numpy as np
import pytest

import oracle
from paper_2604_27325_amd import workloads
from tests.parity import compare_batch

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2604_27325_amd as bed  # noqa: E402


def reference(A):
    """The oracle; LAPACK for a matrix whose oracle vectors are not orthonormal
    (it loses them on the all-ones matrix of order 32)."""
    lam, Q, _ = oracle.syevd(A)
    for b in range(A.shape[0]):
        if np.linalg.norm(Q[b].T @ Q[b] - np.eye(A.shape[1])) > 1e-10:
            lam[b], Q[b] = np.linalg.eigh(A[b])
    return lam, Q


def check(A_np, label, tune=None):
    A_np = np.ascontiguousarray(A_np, dtype=np.float32)
    b, n = A_np.shape[0], A_np.shape[1]
    print(f"[{label}] batch {b} n={n}", flush=True)
    A = torch.from_numpy(A_np).cuda()
    lam = torch.empty(b * n, device="cuda")
    Q = torch.empty(b * n * n, device="cuda")
    info = torch.empty(b, dtype=torch.int32, device="cuda")
    bed.Plan(torch.float32, [n] * b, tune=tune).run(A.view(-1), lam, Q, info)
    vals = bed.syevals(A)
    torch.cuda.synchronize()
    lam_o, Q_o = reference(A_np.astype(np.float64))
    worst, fails = compare_batch(A_np, lam.view(b, n).cpu().numpy(),
                                 Q.view(b, n, n).cpu().numpy(), lam_o, Q_o, np.float32,
                                 info=info.cpu().numpy())
    print(f"  worst {worst}", flush=True)
    assert not fails, f"{label}: {len(fails)} failing, first {fails[:2]}"
    nrm = np.abs(lam_o).max(axis=1).clip(1e-300)
    err = np.abs(vals.cpu().numpy() - lam_o).max(axis=1) / nrm
    assert err.max() <= 1e-5, f"{label}: eigenvalues only {err.max()}"


@pytest.mark.parametrize("n", [1, 2, 3, 7, 8, 9, 15, 16, 17, 24, 25, 31, 32, 33, 40, 41, 48, 49, 63, 64])
def test_sizes(n):
    rng = np.random.default_rng(9000 + n)
    check(np.concatenate([workloads.gaussian_sym(rng, 6, n), workloads.covariance(rng, 6, n)]),
          f"sizes n={n}")


@pytest.mark.parametrize("n", [5, 16, 27, 32, 50, 64])
@pytest.mark.parametrize("mid,big", [(256, 256), (128, 512)])
def test_split_and_degenerate_spectra(n, mid, big):
    """Diagonal, zero, identity, block-diagonal, rank-deficient and graded
    matrices, a Wilkinson matrix and two glued copies of it, tridiagonal
    Toeplitz (both coupling signs)."""
    rng = np.random.default_rng(9100 + n)
    off = np.ones(n - 1)
    wil = np.diag(np.abs(np.arange(n) - (n - 1) / 2.0)) + np.diag(off, 1) + np.diag(off, -1)
    glued = wil.copy()
    h = n // 2
    glued[h - 1, h] = glued[h, h - 1] = 1e-7
    blk = workloads.gaussian_sym(rng, 1, n)[0]
    blk[:h, h:] = blk[h:, :h] = 0.0
    u = rng.standard_normal((n, 2))
    V, _ = np.linalg.qr(rng.standard_normal((n, n)))
    graded = (V * 10.0 ** -np.linspace(0, 6, n)) @ V.T
    mats = [np.diag(np.arange(n) - 2.0), np.zeros((n, n)), np.eye(n) * 3.0, blk, u @ u.T,
            0.5 * (graded + graded.T), wil, glued,
            2 * np.eye(n) + 0.5 * (np.diag(off, 1) + np.diag(off, -1)),
            np.diag(off, 1) * -1.0 + np.diag(off, -1) * -1.0, np.ones((n, n))]
    check(np.stack(mats), f"degenerate n={n}", tune={"threads_mid": mid, "threads_big": big})


@pytest.mark.parametrize("gap", [1e-5, 1e-6, 1e-7, 1e-8, 4e-9, 1e-9, 1e-11])
@pytest.mark.parametrize("n", [16, 32, 64])
def test_close_pairs(n, gap):
    """A 2 x 2 block whose eigenvalues differ by 2 gap, decoupled from the rest
    up to a permutation (so that the stored binary32 matrix keeps the gap)."""
    rng = np.random.default_rng(9200 + n)
    A = workloads.gaussian_sym(rng, 8, n) / np.sqrt(n)
    p, q = n // 3, n // 2
    for M in A:
        M[[p, q], :] = 0.0
        M[:, [p, q]] = 0.0
        M[p, p] = M[q, q] = 0.25
        M[p, q] = M[q, p] = gap
    check(A, f"pair {gap} n={n}")


@pytest.mark.parametrize("n", [8, 16, 20, 32, 47, 64])
@pytest.mark.parametrize("mid,big", [(256, 256), (128, 512)])
def test_decoupled_blocks_that_share_eigenvalues(n, mid, big):
    """Two decoupled blocks with common eigenvalues up to binary32 rounding or a
    planted distance: each vector's twist has to lie in its own block."""
    check(workloads.decoupled_pairs(np.random.default_rng(9300 + n), 48, n),
          f"decoupled n={n}", tune={"threads_mid": mid, "threads_big": big})


def _multiple(rng, n):
    """Twofold and fourfold eigenvalues throughout, one eigenvalue repeated twice and
    six times, cells of the first grid with two apart eigenvalues each, and a pair
    in a decoupled 2 x 2 block, exact and 1e-11 apart."""
    def rotated(w):
        V, _ = np.linalg.qr(rng.standard_normal((n, n)))
        return (V * np.sort(w)) @ V.T

    lin = np.linspace(-1.0, 1.0, n)
    two, six = lin.copy(), lin.copy()
    two[n // 2] = two[n // 2 - 1]
    six[n // 3:n // 3 + 6] = six[n // 3]
    mats = [rotated(np.repeat(lin, 2)[:n]), rotated(np.repeat(lin, 4)[:n]), rotated(two), rotated(six),
            rotated(np.repeat(np.linspace(-1.0, 1.0, (n + 1) // 2), 2)[:n] + 1e-3 * (np.arange(n) % 2))]
    for d in (0.0, 1e-11):
        A = rotated(lin)
        A[[0, n - 1], :] = 0.0
        A[:, [0, n - 1]] = 0.0
        A[0, 0] = A[n - 1, n - 1] = 0.25
        A[0, n - 1] = A[n - 1, 0] = d
        mats.append(A)
    return np.stack(mats)


@pytest.mark.parametrize("n", [8, 15, 16, 24, 31, 32, 33, 39, 40, 48, 64])
@pytest.mark.parametrize("mid,big", [(256, 256), (128, 512)])
def test_multiple_eigenvalues(n, mid, big):
    check(_multiple(np.random.default_rng(9310 + n), n), f"multiple n={n}",
          tune={"threads_mid": mid, "threads_big": big})


@pytest.mark.parametrize("link", [(-13, -9), (-9, -5)])
@pytest.mark.parametrize("n", [8, 16, 32, 47, 64])
def test_weakly_coupled_blocks_that_share_eigenvalues(n, link):
    check(workloads.decoupled_pairs(np.random.default_rng(9320 + n), 48, n, link),
          f"linked {link} n={n}")


@pytest.mark.parametrize("n", [8, 16, 24, 32, 48, 64, 96, 128])
def test_eigenvalues_alone_of_null_and_repeated_blocks(n):
    """Small determinants: null blocks of half, three quarters and all of the matrix
    but one row, low rank, and exact copies of small blocks; ascending."""
    rng = np.random.default_rng(9330 + n)
    mats = []
    for m in (n // 2, n // 4, 1):
        A = np.zeros((n, n))
        A[:m, :m] = workloads.gaussian_sym(rng, 1, m)[0]
        mats.append(A)
        X = rng.standard_normal((m, n))
        mats.append(X.T @ X)
    for k in (2, 4, 8):
        L = 2.0 * np.eye(k) - np.eye(k, k=1) - np.eye(k, k=-1)
        mats += [np.kron(L, np.eye(n // k)), np.kron(np.eye(n // k), L)]
    A = np.stack(mats).astype(np.float32)
    vals = bed.syevals(torch.from_numpy(A).cuda()).cpu().numpy()
    ref = np.linalg.eigvalsh(A.astype(np.float64))
    assert np.isfinite(vals).all() and (np.diff(vals, axis=1) >= 0).all()
    assert (np.abs(vals - ref).max(axis=1) <= 1e-5 * np.abs(ref).max(axis=1)).all()


@pytest.mark.parametrize("n", [16, 24, 32, 48, 64])
def test_graded_spectra_and_many_close_pairs(n):
    """Eigenvalues over four decades (crowded at one end of the first grid), and two to
    nine close pairs or runs."""
    rng = np.random.default_rng(9340 + n)
    mats = []
    for t in range(24):
        w = np.sort(10.0 ** rng.uniform(-4.0, 0.0, n))
        k = min(2 + t // 3, n // 2)
        if t % 3 == 1:
            w[1:2 * k:2] = w[:2 * k:2] * (1.0 + 1e-7)
        elif t % 3 == 2:
            w[n - k:] = 1.0 + 1e-8 * np.arange(k)
        V, _ = np.linalg.qr(rng.standard_normal((n, n)))
        mats.append((V * w) @ V.T)
    check(np.stack(mats), f"graded n={n}")


@pytest.mark.parametrize("n", [16, 32, 33, 64])
def test_clusters_and_runs_of_close_eigenvalues(n):
    """Neighbouring cells of the first grid full (two clusters, a spike beside a narrow
    bulk), pairs at random places, and runs of up to twenty close eigenvalues."""
    rng = np.random.default_rng(9350 + n)
    mats = []
    for t in range(20):
        h = n // 2
        if t % 4 == 0:
            w = np.concatenate([rng.uniform(0.0, 0.02, h), rng.uniform(1.0, 1.02, n - h)])
        elif t % 4 == 1:
            w = np.concatenate([rng.uniform(0.25, 2.25, n - 1), [10.0 ** (1 + t / 5)]])
        elif t % 4 == 2:
            w = np.repeat(rng.uniform(-1.0, 1.0, (n + 1) // 2), 2)[:n]
        else:
            w = rng.uniform(-1.0, 1.0, n)
            k = min(t, n - 2)
            w[:k] = w[0] + 1e-7 * np.arange(k)
        V, _ = np.linalg.qr(rng.standard_normal((n, n)))
        mats.append((V * w) @ V.T)
    check(np.stack(mats), f"clusters n={n}")
