"""Continuous-batching server: results in a mix are bitwise equal to solo
solves and within the parity rules of the binary64 oracle; admission refuses
by in-flight matrices and by memory; a request submitted right after the
asynchronous work that produces its input reads the finished input; latency
and throughput are reported."""
import time

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

DEV = torch.device("cuda:0")
# bounded spin that keeps a producer stream busy for a few milliseconds
SPIN_CYCLES = 20_000_000


def make_requests(count, seed=5000, cmax=64):
    arr, counts, ns = workloads.serving_trace(seed=seed, requests=count, qps=5000.0, cmax=cmax)
    reqs = []
    for i in range(count):
        A = torch.from_numpy(workloads.serving_matrices(seed + 1 + i, int(counts[i]), int(ns[i])))
        reqs.append(A.to(DEV))
    return reqs


def test_mixed_results_equal_solo_and_match_oracle():
    reqs = make_requests(60)
    solo = [bed.syevd(A) for A in reqs]
    torch.cuda.synchronize()
    srv = bed.Server(streams=4)
    outs, tickets = [], []
    for A in reqs:
        lam = torch.empty(A.shape[0], A.shape[1], device=DEV)
        Q = torch.empty_like(A)
        info = torch.empty(A.shape[0], dtype=torch.int32, device=DEV)
        tk = srv.submit(A, lam, Q, info)
        assert tk is not None
        outs.append((lam, Q, info))
        tickets.append(tk)
    srv.drain()
    As, lg, qg, infos = [], [], [], []
    for tk, (lam, Q, info), (lam_s, Q_s), A in zip(tickets, outs, solo, reqs):
        done, lat = srv.poll(tk)
        assert done and lat > 0
        assert torch.equal(lam, lam_s) and torch.equal(Q, Q_s)
        As += list(A.cpu().numpy())
        lg += list(lam.cpu().numpy())
        qg += list(Q.cpu().numpy())
        infos += list(info.cpu().numpy())
    srv.close()
    # every served matrix against the oracle (grouped by size for the oracle call)
    lo, qo = [None] * len(As), [None] * len(As)
    by_n = {}
    for i, M in enumerate(As):
        by_n.setdefault(M.shape[0], []).append(i)
    for n, idx in by_n.items():
        l_o, q_o, _ = oracle.syevd(np.stack([As[i] for i in idx]).astype(np.float64))
        for j, i in enumerate(idx):
            lo[i], qo[i] = l_o[j], q_o[j]
    worst, fails = compare_batch(As, lg, qg, lo, qo, np.float32, info=np.array(infos))
    print(f"[serving vs oracle] {len(As)} matrices, worst {worst}", flush=True)
    assert not fails, fails[:3]


def test_admission_refuses_by_inflight_limit_then_admits():
    """The first request waits on a producer stream kept busy by a bounded spin,
    so it is certainly still in flight when the second is submitted."""
    reqs = make_requests(2, seed=6000)
    n0 = reqs[0].shape[0]
    # each request fits alone, both together do not
    srv = bed.Server(streams=1, max_inflight=max(n0, reqs[1].shape[0]))
    lam = torch.empty(n0, reqs[0].shape[1], device=DEV)
    Q = torch.empty_like(reqs[0])
    prod = torch.cuda.Stream()
    prod.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(prod):
        torch.cuda._sleep(SPIN_CYCLES)
    first = srv.submit(reqs[0], lam, Q, stream=prod)
    assert first is not None
    lam2 = torch.empty(reqs[1].shape[0], reqs[1].shape[1], device=DEV)
    Q2 = torch.empty_like(reqs[1])
    assert srv.submit(reqs[1], lam2, Q2) is None  # in-flight limit reached
    srv.drain()
    second = srv.submit(reqs[1], lam2, Q2)  # admitted once the first completed
    assert second is not None
    srv.drain()
    l1, q1 = bed.syevd(reqs[0])
    l2, q2 = bed.syevd(reqs[1])
    assert torch.equal(lam, l1) and torch.equal(Q, q1)
    assert torch.equal(lam2, l2) and torch.equal(Q2, q2)
    srv.close()


def test_admission_refuses_by_memory_budget():
    reqs = make_requests(3, seed=6100)
    A = reqs[2]
    need = A.shape[0] * (2 * A.shape[1] ** 2 + A.shape[1]) * 4  # A, Q and lambda bytes
    tiny = bed.Server(streams=2, mem_budget=need - 1)
    assert tiny.submit(A, torch.empty(A.shape[:2], device=DEV), torch.empty_like(A)) is None
    tiny.close()
    exact = bed.Server(streams=2, mem_budget=need)
    lam, Q = torch.empty(A.shape[:2], device=DEV), torch.empty_like(A)
    assert exact.submit(A, lam, Q) is not None
    exact.drain()
    l_s, q_s = bed.syevd(A)
    assert torch.equal(lam, l_s) and torch.equal(Q, q_s)
    exact.close()


def test_submit_right_after_async_producer():
    """A is produced by kernels still queued on the submitting stream (behind a
    bounded spin): the request's step waits for them, so it solves the final A,
    with no host synchronization in between."""
    reqs = make_requests(4, seed=6200)
    srv = bed.Server(streams=2)
    prod = torch.cuda.Stream()
    prod.wait_stream(torch.cuda.current_stream())
    outs = []
    for src in reqs:
        with torch.cuda.stream(prod):
            A = torch.zeros_like(src)
            torch.cuda._sleep(SPIN_CYCLES // 4)
            A.copy_(src)  # the input appears only after the spin
        lam, Q = torch.empty(src.shape[:2], device=DEV), torch.empty_like(src)
        tk = srv.submit(A, lam, Q, stream=prod)
        assert tk is not None
        outs.append((A, lam, Q))
    srv.drain()
    torch.cuda.synchronize()
    for src, (A, lam, Q) in zip(reqs, outs):
        l_s, q_s = bed.syevd(src)
        assert torch.equal(lam, l_s) and torch.equal(Q, q_s)
    srv.close()


def test_latency_and_throughput_reported():
    reqs = make_requests(200, seed=7000)
    outs = [(torch.empty(A.shape[0], A.shape[1], device=DEV), torch.empty_like(A)) for A in reqs]
    torch.cuda.synchronize()
    srv = bed.Server(streams=4)
    t0 = time.perf_counter()
    tickets = [srv.submit(A, o[0], o[1]) for A, o in zip(reqs, outs)]
    srv.drain()
    el = time.perf_counter() - t0
    lats = np.array([srv.poll(tk)[1] for tk in tickets])
    srv.close()
    mats = sum(A.shape[0] for A in reqs)
    print(f"[serving] {mats / el:.0f} matrices/s p50 {np.percentile(lats, 50):.0f} us "
          f"p99 {np.percentile(lats, 99):.0f} us", flush=True)
    assert np.all(lats > 0)


def test_requests_from_two_threads():
    """Two threads submit from streams of their own while the scheduler launches: every
    request's result is that of a solo solve."""
    import threading
    reqs = make_requests(80, seed=8000)
    solo = [bed.syevd(A) for A in reqs]
    torch.cuda.synchronize()
    srv = bed.Server(streams=3, max_step=64)
    outs = [(torch.empty(A.shape[0], A.shape[1], device=DEV), torch.empty_like(A)) for A in reqs]
    tickets, errors = [None] * len(reqs), []
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()

    def submit(k):
        try:
            for i in range(k, len(reqs), 2):
                tickets[i] = srv.submit(reqs[i], *outs[i], stream=streams[k])
        except Exception as e:  # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=submit, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not errors and None not in tickets
    srv.drain()
    assert len(set(tickets)) == len(reqs)
    for tk, (lam, Q), (lam_s, Q_s) in zip(tickets, outs, solo):
        assert srv.poll(tk)[0]
        assert torch.equal(lam, lam_s) and torch.equal(Q, Q_s)
    srv.close()
