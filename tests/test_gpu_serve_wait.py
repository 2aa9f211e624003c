"""A waiting poll of the serving loop: it returns with the first batch that is
done, whichever slot it is in, and leaves the core to others while it waits.
The batches are long because one wave searches all their queries in turn
(launch_waves = 1)."""
import time

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2402_11354_amd")

pytestmark = pytest.mark.gpu

SMALL = W.Workload("serve_wait_4k_d64", 4000, 400, 64, 16, 32, 4, 16, W.ANGULAR, "sphere500", 0.1, 10, 32, 1006)


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(torch.device("cuda:0"))


@pytest.fixture(scope="module")
def case():
    w = SMALL
    x, q = W.make_base(w), W.make_queries(w)
    g, entry = W.build_graph(x, w.R, w.cand)
    A, B = W.directions_for(w)
    return q, P.peos_build_tables(T(x), T(g), entry, w.L, w.m, T(A), T(B), w.metric)


def test_first_batch_done_is_returned(case):
    q, index = case
    srv = P.Server(index, max_batch=400, max_k=10, max_ef=256, max_inflight=2, pool=1, launch_waves=1)
    try:
        for _ in range(2):  # (the first round warms the kernels up)
            long_t = srv.submit(q, 10, 256)
            short_t = srv.submit(q[:1], 10, 16)
            done = srv.poll(wait=True)
            c = srv.counters()
            got = [t for t, _, _ in done]
            print("[gpu] first poll:", got, c, flush=True)
            first = got == [short_t] and c["inflight"] == 1
            while srv.live:
                done += srv.poll(wait=True)
            assert sorted(t for t, _, _ in done) == [long_t, short_t]
        assert first
    finally:
        srv.close()


@pytest.mark.parametrize("batches", [1, 2])
def test_waiting_leaves_the_core(case, batches):
    q, index = case
    srv = P.Server(index, max_batch=400, max_k=10, max_ef=256, max_inflight=batches, pool=1, launch_waves=1)
    try:
        for _ in range(2):
            for _ in range(batches):
                srv.submit(q, 10, 256)
            wall, cpu = time.perf_counter(), time.thread_time()
            srv.poll(wait=True)
            wall, cpu = time.perf_counter() - wall, time.thread_time() - cpu
            print(f"[gpu] {batches} in flight: waited {wall * 1e3:.1f} ms, of these {cpu * 1e3:.1f} ms on the core",
                  flush=True)
            while srv.live:
                srv.poll(wait=True)
        assert wall > 10e-3  # a wait worth the name
        assert cpu < 0.5 * wall
    finally:
        srv.close()
