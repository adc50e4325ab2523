"""GPU parity of the forward solve against the binary64 oracle (through the
C-ABI library).  Inputs are seeded synthetic workloads; expected values come
from the oracle at test time."""
import numpy as np
import pytest

import oracle
from paper_2604_27325_amd import workloads
from tests.parity import compare_batch

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, skipped there
    pytest.skip("no GPU", allow_module_level=True)

import paper_2604_27325_amd as bed  # noqa: E402

DEV = torch.device("cuda:0")


def run_gpu(A_np):
    A = torch.from_numpy(np.ascontiguousarray(A_np)).to(DEV)
    lam, Q, info = bed.syevd(A, return_info=True)
    torch.cuda.synchronize()
    return lam.cpu().numpy(), Q.cpu().numpy(), info.cpu().numpy()


def check(A_np, label):
    dtype = np.float32 if A_np.dtype == np.float32 else np.float64
    lam_g, Q_g, info = run_gpu(A_np)
    lam_o, Q_o, info_o = oracle.syevd(A_np.astype(np.float64))
    worst, fails = compare_batch(A_np, lam_g, Q_g, lam_o, Q_o, dtype, info=info)
    print(f"[{label}] worst {worst}", flush=True)
    assert not fails, f"{label}: {len(fails)} failing matrices, first {fails[:3]}"
    return worst


def test_plain_fp64_batch64_n16():
    check(workloads.plain_fp64(), "plain fp64 64x16")


@pytest.mark.parametrize("n", [32, 48, 64])
def test_paper_scale_fp32_batch512(n):
    A, planted, _ = workloads.paper_scale(n)
    check(A, f"paper scale n={n}")


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 9, 15, 16, 17, 23, 24, 31, 32, 33, 40, 47, 63, 64])
@pytest.mark.parametrize("dt", [np.float32, np.float64])
def test_every_size_class_and_ragged_tail(n, dt):
    rng = np.random.default_rng(500 + n)
    A = np.concatenate([workloads.gaussian_sym(rng, 6, n), workloads.covariance(rng, 6, n)])
    check(A.astype(dt), f"n={n} {dt.__name__}")


@pytest.mark.parametrize("dt", [np.float32, np.float64])
def test_structured_matrices(dt):
    n = 37
    rng = np.random.default_rng(9)
    u = rng.standard_normal(n)
    mats = [np.diag(rng.permutation(np.arange(n, dtype=np.float64))),
            np.eye(n) * 3.0,
            np.zeros((n, n)),
            np.outer(u, u),
            np.diag(np.full(n, 0.5)) + np.diag(np.full(n - 1, -0.3), 1) + np.diag(np.full(n - 1, -0.3), -1)]
    for i, M in enumerate(mats):
        check(M[None].astype(dt), f"structured {i} {dt.__name__}")


def test_nonfinite_input_reports_info_minus_one():
    rng = np.random.default_rng(3)
    A = workloads.gaussian_sym(rng, 4, 20).astype(np.float32)
    A[1, 5, 2] = np.nan     # lower triangle: detected
    A[2, 3, 9] = np.inf     # upper triangle: never read
    lam, Q, info = run_gpu(A)
    assert list(info) == [0, -1, 0, 0]
    assert np.all(np.isnan(lam[1])) and np.all(np.isnan(Q[1]))
    lam_o, Q_o, _ = oracle.syevd(np.tril(A[2]).astype(np.float64))
    assert np.abs(lam[2] - lam_o).max() < 1e-5 * np.abs(lam_o).max()


def test_in_place_and_determinism():
    rng = np.random.default_rng(4)
    A_np = workloads.gaussian_sym(rng, 64, 64).astype(np.float32)
    A = torch.from_numpy(A_np).to(DEV)
    lam1, Q1 = bed.syevd(A)
    lam2, Q2 = bed.syevd(A)
    assert torch.equal(lam1, lam2) and torch.equal(Q1, Q2)  # bitwise repeatable
    B = A.clone()
    lam3 = torch.empty(64, 64, device=DEV)
    bed.syevd_packed([64] * 64, B.view(-1), lam=lam3.view(-1), Q=B.view(-1))  # Q == A
    assert torch.equal(lam3, lam1) and torch.equal(B, Q1)


@pytest.mark.parametrize("n", [1, 2, 3, 5, 9, 16, 17, 31, 32, 33, 48, 63, 64])
@pytest.mark.parametrize("dt", [np.float32, np.float64])
def test_eigenvalues_only_matches_oracle(n, dt):
    """bed_syevals (no eigenvectors: only the end rows of every node's block
    are carried between depths) against the oracle's eigenvalues (R1), on
    Gaussian and covariance matrices and on the planted-pair workload."""
    rng = np.random.default_rng(5 + n)
    A_np = np.concatenate([workloads.gaussian_sym(rng, 16, n), workloads.covariance(rng, 16, n)])
    if n in (32, 48, 64):
        A_np = np.concatenate([A_np, workloads.paper_scale(n)[0][:64]])
    A_np = A_np.astype(dt)
    A = torch.from_numpy(A_np).to(DEV)
    lam, _, info = bed.syevd_packed([n] * A_np.shape[0], A.view(-1), want_vectors=False)
    lam = lam.view(-1, n).cpu().numpy()
    lam_o, _, _ = oracle.syevd(A_np.astype(np.float64))
    worst, fails = compare_batch(A_np, lam, None, lam_o, None, dt, info=info.cpu().numpy())
    print(f"[syevals n={n} {dt.__name__}] worst {worst}", flush=True)
    assert not fails, fails[:3]


def test_eigenvalues_only_uneven_packed_batch():
    ns, mats = workloads.uneven(batch=300)
    _, flat = workloads.pack(mats)
    lam, _, info = bed.syevd_packed(ns, torch.from_numpy(flat).to(DEV), want_vectors=False)
    lam, info = lam.cpu().numpy(), info.cpu().numpy()
    lam_o, _, _ = oracle.syevd_packed(ns, flat.astype(np.float64))
    offs = np.concatenate([[0], np.cumsum(ns)])
    lg = [lam[offs[i]:offs[i + 1]] for i in range(len(ns))]
    lo = [lam_o[offs[i]:offs[i + 1]] for i in range(len(ns))]
    worst, fails = compare_batch(mats, lg, None, lo, None, np.float32, info=info)
    print(f"[syevals uneven] worst {worst}", flush=True)
    assert not fails, fails[:3]


def test_uneven_packed_batch_matches_oracle():
    ns, mats = workloads.uneven(batch=300)
    ns_, flat = workloads.pack(mats)
    A = torch.from_numpy(flat).to(DEV)
    lam, Q, info = bed.syevd_packed(ns, A)
    torch.cuda.synchronize()
    lam, Q, info = lam.cpu().numpy(), Q.cpu().numpy(), info.cpu().numpy()
    lam_o, Q_o, _ = oracle.syevd_packed(ns, flat.astype(np.float64))
    offA = offL = 0
    As, lg, qg, lo, qo = [], [], [], [], []
    for n in ns:
        As.append(mats[len(As)])
        lg.append(lam[offL:offL + n]); lo.append(lam_o[offL:offL + n])
        qg.append(Q[offA:offA + n * n].reshape(n, n)); qo.append(Q_o[offA:offA + n * n].reshape(n, n))
        offA += n * n
        offL += n
    worst, fails = compare_batch(As, lg, qg, lo, qo, np.float32, info=info)
    print("[uneven]", worst)
    assert not fails, fails[:3]


def test_batch_zero_is_noop():
    A = torch.empty(0, device=DEV)
    lam, Q, info = bed.syevd_packed([], A)
    assert lam.numel() == 0 and Q.numel() == 0


@pytest.mark.parametrize("dt", [np.float32, np.float64])
def test_scaled_and_block_structured_matrices(dt):
    """Scale invariance (every threshold is relative) at sizes that are a single
    leaf, one merge, ragged and full; block-diagonal input (zero couplings in
    the tridiagonal form, exactly repeated eigenvalues from repeated blocks);
    Wilkinson's W21+ (pairs agreeing to many digits)."""
    rng = np.random.default_rng(77)
    s_hi, s_lo = (1e12, 1e-12) if dt == np.float32 else (1e100, 1e-100)
    mats = []
    for n in (4, 5, 8, 37, 64):
        G = workloads.gaussian_sym(rng, 1, n)[0]
        mats += [G * s_hi, G * s_lo]
    blk = workloads.gaussian_sym(rng, 1, 4)[0]
    B = np.zeros((24, 24))
    for b in range(6):
        B[4 * b:4 * b + 4, 4 * b:4 * b + 4] = blk if b % 2 == 0 else workloads.gaussian_sym(rng, 1, 4)[0]
    mats.append(B)
    W = np.diag(np.abs(np.arange(-10.0, 11.0))) + np.diag(np.ones(20), 1) + np.diag(np.ones(20), -1)
    mats.append(W)
    for i, M in enumerate(mats):
        check(M[None].astype(dt), f"scaled/block {i} n={M.shape[0]} {dt.__name__}")


def _null_blocks(rng, batch, n):
    """Graph Laplacians (weighted or not) and 0/1/-1 matrices so sparse that many
    rows are empty, zero but for a few rows and columns, and diagonal blocks with
    scales 1, 1e-10, 1e-20 and 1e-30."""
    out = []
    for t in range(batch):
        W = np.triu(rng.uniform(size=(n, n)) < rng.uniform(0.5, 3.0) / n, 1).astype(np.float64)
        if t % 4 == 0:
            W *= rng.uniform(0.0, 1.0, (n, n)).astype(np.float32)
        if t % 4 < 2:
            A = np.diag((W + W.T).sum(axis=1)) - W - W.T
        elif t % 4 == 2:
            W *= rng.integers(-1, 2, (n, n))
            A = W + W.T + np.diag(rng.integers(-1, 2, n) * (rng.uniform(size=n) < 0.3))
        else:
            s = np.repeat(10.0 ** (-10.0 * np.arange(4)), (n + 3) // 4)[:n]
            A = np.where(s[:, None] == s[None, :], workloads.gaussian_sym(rng, 1, n)[0] * s, 0.0)
        out.append(A)
    return np.stack(out)


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("n", [5, 11, 16, 17, 22, 32, 40, 64, 65, 96, 128])
def test_null_blocks(dt, n):
    """Matrices with empty rows: the reduction leaves rounding's rounding in the
    null block, whose merges are as far below the matrix's scale."""
    if dt == np.float64 and n > 64:
        pytest.skip("binary32 only above 64")
    A = _null_blocks(np.random.default_rng(7700 + n), 64, n).astype(dt)
    At = torch.from_numpy(A).cuda()
    lam, Q, info = bed.syevd(At, return_info=True)
    vals = bed.syevals(At).cpu().numpy()
    lam, Q = lam.cpu().numpy(), Q.double().cpu().numpy()
    A = A.astype(np.float64)
    ref = np.linalg.eigvalsh(A)
    nrm = np.abs(ref).max(axis=1).clip(1e-30)
    tol_lam, tol = (1e-5, 1e-5) if dt == np.float32 else (1e-12, 1e-13)
    assert not info.cpu().numpy().any()
    for got in (lam, vals):
        assert np.isfinite(got).all() and (np.diff(got, axis=1) >= 0).all()
        assert (np.abs(got - ref).max(axis=1) <= tol_lam * nrm).all()
    assert np.isfinite(Q).all()
    res = np.linalg.norm(A @ Q - Q * lam[:, None, :], axis=(1, 2)) / \
        np.linalg.norm(A, axis=(1, 2)).clip(1e-30)
    orth = np.linalg.norm(np.swapaxes(Q, 1, 2) @ Q - np.eye(n), axis=(1, 2))
    assert res.max() <= tol and orth.max() <= tol, (res.max(), orth.max())
