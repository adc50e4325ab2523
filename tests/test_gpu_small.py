"""Uniform batches of order n <= 4 (one lane per matrix): both storage types, at
the edges of a wave, in place, at addresses that rule out wide accesses, with
degenerate, scaled and non-finite matrices."""
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

NP = {torch.float32: np.float32, torch.float64: np.float64}


def inputs(n, batch, seed):
    rng = np.random.default_rng(seed)
    A = workloads.gaussian_sym(rng, batch, n)
    if batch >= 8:
        A[0] = 0.0
        A[1] = np.eye(n) * 2.5
        A[2] = np.diag(np.arange(n, 0, -1.0))
        A[3] = 1.0
        A[4] = np.outer(np.arange(1, n + 1), np.arange(1, n + 1))
        A[5] *= 1e-30
        A[6] *= 1e30
        A[7] = np.diag(np.full(n, 0.5)) + 1e-7 * A[7]
    return A


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [1, 2, 3, 4])
@pytest.mark.parametrize("batch,shift", [(1, 0), (63, 1), (64, 0), (65, 3), (1000, 0)])
def test_small_orders(dtype, n, batch, shift):
    A_np = inputs(n, batch, 700 + n).astype(NP[dtype])
    print(f"[small n={n} {dtype} batch {batch} shift {shift}]", flush=True)

    def at(numel):  # a buffer `shift` elements past an aligned address
        return torch.empty(numel + shift, dtype=dtype, device="cuda")[shift:]

    A, lam, Q = at(batch * n * n), at(batch * n), at(batch * n * n)
    A.copy_(torch.from_numpy(A_np.ravel()))
    info = torch.full((batch,), 7, dtype=torch.int32, device="cuda")
    bed.syevd_packed([n] * batch, A, lam=lam, Q=Q, info=info)
    vals = bed.syevals(A.view(batch, n, n))
    lam_o, Q_o, _ = oracle.syevd(A_np.astype(np.float64))
    worst, fails = compare_batch(A_np, lam.view(batch, n).cpu().numpy(),
                                 Q.view(batch, n, n).cpu().numpy(), lam_o, Q_o, NP[dtype],
                                 info=info.cpu().numpy())
    assert not fails, (worst, fails[:3])
    assert torch.equal(vals.view(-1), lam)
    inplace = A.clone()
    bed.syevd_packed([n] * batch, inplace, lam=lam, Q=inplace, info=info)
    assert torch.equal(inplace, Q)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [1, 3, 4])
def test_small_nonfinite(dtype, n):
    A_np = inputs(n, 70, 710 + n)
    A_np[5, n - 1, 0] = np.nan
    A_np[66, 0, 0] = np.inf
    if n > 1:
        A_np[9, 0, n - 1] = np.nan  # upper triangle: not read
    A = torch.from_numpy(A_np).to("cuda", dtype)
    lam, Q, info = bed.syevd(A, return_info=True)
    info = info.cpu().numpy()
    assert info[5] == -1 and info[66] == -1 and np.count_nonzero(info) == 2
    assert bool(torch.isnan(lam[5]).all()) and bool(torch.isnan(Q[66]).all())
    keep = np.ones(70, bool)
    keep[[5, 66]] = False
    assert bool(torch.isfinite(Q[torch.from_numpy(keep).cuda()]).all())


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [2, 3, 4])
def test_small_in_place_over_many_workgroups(dtype, n):
    """Q == A with a partly filled last wave: its idle lanes stay off the matrices
    that other workgroups overwrite, so every run gives the out-of-place bits."""
    batch = 64 * 300 + 5
    A_np = workloads.gaussian_sym(np.random.default_rng(720 + n), batch, n).astype(NP[dtype])
    A = torch.from_numpy(A_np).cuda().view(-1)
    lam = torch.empty(batch * n, dtype=dtype, device="cuda")
    lam0, Q0, _ = bed.syevd_packed([n] * batch, A)
    for _ in range(20):
        inplace = A.clone()
        bed.syevd_packed([n] * batch, inplace, lam=lam, Q=inplace)
        assert torch.equal(inplace, Q0) and torch.equal(lam, lam0)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [2, 3, 4])
def test_small_results_do_not_depend_on_the_batch(dtype, n):
    """Each matrix of a wave gives the same bits alone, beside others that take
    fewer or more Jacobi sweeps, and in another place."""
    rng = np.random.default_rng(730 + n)
    A_np = workloads.gaussian_sym(rng, 256, n)
    A_np[::3] = 1e-5 * A_np[::3] + np.diag(np.arange(n) + 1.0)  # one or two sweeps
    A = torch.from_numpy(A_np).to("cuda", dtype)
    lam, Q = bed.syevd(A)
    perm = torch.from_numpy(rng.permutation(256)).cuda()
    lam_p, Q_p = bed.syevd(A[perm].contiguous())
    assert torch.equal(lam_p, lam[perm]) and torch.equal(Q_p, Q[perm])
    for i in range(0, 256, 5):
        lam_1, Q_1 = bed.syevd(A[i:i + 1])
        assert torch.equal(lam_1[0], lam[i]) and torch.equal(Q_1[0], Q[i]), i
