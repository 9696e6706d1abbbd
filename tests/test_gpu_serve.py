"""The queue-driven serving session (resident kernel, Section 4.2.3) against vf_search: every job's result equals
the batched search of the same query; the kernel ends by itself when its bounded wait expires."""
import time

import numpy as np
import pytest

from paper_2506_00812_amd.workloads import make_workload
from tests.gpu_util import assert_close_with_ties, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vf():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2506_00812_amd import binding
    binding.load_library()
    return binding


def _wait(server, jobs, timeout_s=60.0):
    out, t0 = {}, time.time()
    pending = list(jobs)
    while pending:
        assert time.time() - t0 < timeout_s, f"{len(pending)} jobs still pending"
        rest = []
        for j in pending:
            r = server.poll(j)
            if r is None:
                rest.append(j)
            else:
                out[j] = r
        pending = rest
    return out


def _labels_with_and(w, nq, rng):
    first = w.qlabel_ids[w.qlabel_offsets[:-1]][:nq]
    labs = []
    for j in range(nq):
        if j % 3 == 0:
            labs.append([int(first[j]), int(rng.integers(0, min(8, w.spec.n_labels)))])
        else:
            labs.append([int(first[j])])
    return labs


@pytest.mark.parametrize("name", ["uint8", "float32", "float32 dim 96"])
def test_served_queries_equal_batched_search(vf, name):
    import torch
    if name == "uint8":
        w = make_workload("tiny", nq=600)
    elif name == "float32":
        w = make_workload("c2", n=30_000, nq=600, n_labels=60, n_clusters=64, T=800, graph_degree=32)
    else:
        w = make_workload("c5", n=20_000, nq=600, n_labels=80, n_clusters=32, T=600, graph_degree=16)
    s = w.spec
    X = torch.from_numpy(w.vectors).cuda()
    Q = torch.from_numpy(w.queries).cuda()
    ix = vf.build_index(X, w.label_offsets, w.label_ids, s.n_labels, s.T, s.graph_degree)
    rng = np.random.default_rng(3)
    nq = 600
    labs = _labels_with_and(w, nq, rng)
    off = np.zeros(nq + 1, dtype=np.int64)
    np.cumsum([len(l) for l in labs], out=off[1:])
    ids = np.concatenate(labs).astype(np.int32)
    params = dict(itopk=32, width=2, iters=8, n_seeds=128)
    ref_i, ref_d = vf.search(ix, Q[:nq], off, ids, 10, **params)
    torch.cuda.synchronize()
    ref_i, ref_d = to_np(ref_i), to_np(ref_d)
    S = ix.export("S")
    smallest = np.array([S[l].min() for l in labs])
    graph = smallest >= s.T
    assert graph.sum() > 100 and (~graph).sum() > 100

    srv = vf.Server(ix, 10, n_workers=64, ring_slots=256, **params)
    try:
        pending, got = [], {}
        for j in range(nq):                                  # more jobs than ring slots: the ring wraps
            job = srv.submit(w.queries[j], labs[j])
            while job is None:                               # ring full: the oldest jobs are still running
                time.sleep(0.001)
                job = srv.submit(w.queries[j], labs[j])
            assert job == j
            pending.append(job)
            if len(pending) >= 192:                          # results must be read before the ring wraps over them
                got.update(_wait(srv, pending[:64]))
                pending = pending[64:]
        got.update(_wait(srv, pending))
        # the same queries once more as one host batch through the session
        ri, rd, lat = srv.run(w.queries[:nq], off, ids, in_flight=48)
        for j in range(nq):
            assert np.array_equal(ri[j], got[j][0]) and np.array_equal(rd[j].view(np.uint32), got[j][1].view(np.uint32))
        assert (lat > 0).all()
    finally:
        done, why = srv.end()
    assert done == 2 * nq and why == 1
    # workers of one and of four waves (the default is eight): the seeds are shared out differently, the bits are the same
    for waves in (1, 4):
        srv = vf.Server(ix, 10, n_workers=32, ring_slots=256, waves_per_worker=waves, **params)
        try:
            wi, wd, _ = srv.run(w.queries[:nq], off, ids, in_flight=32)
        finally:
            done, why = srv.end()
        assert done == nq and why == 1
        assert np.array_equal(wi, ri) and np.array_equal(wd.view(np.uint32), rd.view(np.uint32)), f"{waves} waves per worker"
    gi = np.stack([got[j][0] for j in range(nq)])
    gd = np.stack([got[j][1] for j in range(nq)])
    assert np.array_equal(gi[graph], ref_i[graph]), "graph-searched jobs"
    assert np.array_equal(gd[graph].view(np.uint32), ref_d[graph].view(np.uint32))
    if s.dtype == "uint8":
        assert np.array_equal(gi[~graph], ref_i[~graph]) and np.array_equal(gd[~graph], ref_d[~graph])
    else:
        assert_close_with_ties(gi[~graph], gd[~graph], ref_i[~graph], ref_d[~graph], 1e-4, "scanned jobs")


def test_serving_kernel_ends_by_itself(vf, tiny):
    """Bounded waits: with a small idle bound the kernel leaves on its own, vf_serve_end returns at once and
    reports why; submissions after that are refused; max_jobs ends a session as well."""
    import torch
    s = tiny.spec
    X = torch.from_numpy(tiny.vectors).cuda()
    ix = vf.build_index(X, tiny.label_offsets, tiny.label_ids, s.n_labels, s.T, s.graph_degree)
    srv = vf.Server(ix, 10, itopk=32, width=1, iters=4, n_seeds=64, n_workers=8, ring_slots=16, idle_polls=2000)
    job = srv.submit(tiny.queries[0], [int(tiny.qlabel_ids[0])])
    r = _wait(srv, [job])
    assert (r[job][0] >= 0).any()
    t0 = time.time()
    while time.time() - t0 < 20.0:                           # the idle bound expires within milliseconds
        try:
            if srv.submit(tiny.queries[1], [int(tiny.qlabel_ids[1])]) is None:
                time.sleep(0.01)
                continue
            time.sleep(0.05)
        except vf.VecflowError as e:
            assert "ended" in str(e)
            break
    else:
        pytest.fail("the kernel did not end by itself")
    done, why = srv.end()
    assert why == 3 and done >= 1
    # max_jobs
    srv = vf.Server(ix, 10, itopk=32, width=1, iters=4, n_seeds=64, n_workers=8, ring_slots=16, max_jobs=5)
    jobs = [srv.submit(tiny.queries[j], [int(tiny.qlabel_ids[j])]) for j in range(5)]
    _wait(srv, jobs)
    with pytest.raises(vf.VecflowError):
        srv.submit(tiny.queries[5], [int(tiny.qlabel_ids[5])])
    done, why = srv.end()
    assert done == 5 and why == 2
    # bad arguments never reach the ring
    srv = vf.Server(ix, 10, itopk=32, width=1, iters=4, n_seeds=64, n_workers=4, ring_slots=8, idle_polls=200000)
    with pytest.raises(vf.VecflowError, match="outside"):
        srv.submit(tiny.queries[0], [s.n_labels])
    with pytest.raises(vf.VecflowError, match="1 to 8"):
        srv.submit(tiny.queries[0], list(range(9)))
    assert srv.end() == (0, 1)
    with pytest.raises(vf.VecflowError, match="at most 64"):
        vf.Server(ix, 10, itopk=128, width=1, iters=4, n_seeds=64)


@pytest.mark.parametrize("ring_slots,n_workers,waves,in_flight", [(1, 240, 8, 1), (3, 5, 4, 3), (70, 64, 1, 70), (64, 1, 8, 64), (1024, 1023, 8, 300)])
def test_jobs_are_handed_over_once_each(vf, tiny, ring_slots, n_workers, waves, in_flight):
    """Workers draw job numbers and wait at the slots' ready words: rings with fewer slots than workers, with one slot, more
    jobs published at once than a wave has lanes, one worker for all of them; and a session of the most workers."""
    import torch
    s = tiny.spec
    X = torch.from_numpy(tiny.vectors).cuda()
    ix = vf.build_index(X, tiny.label_offsets, tiny.label_ids, s.n_labels, s.T, s.graph_degree)
    nq = min(300, s.nq)
    params = dict(itopk=32, width=1, iters=6, n_seeds=64)
    off, ids = tiny.qlabel_offsets[:nq + 1], tiny.qlabel_ids[:tiny.qlabel_offsets[nq]]
    ref_i, ref_d = vf.search(ix, torch.from_numpy(tiny.queries[:nq]).cuda(), off, ids, 10, **params)
    srv = vf.Server(ix, 10, n_workers=n_workers, ring_slots=ring_slots, waves_per_worker=waves, **params)
    try:
        for _ in range(2):
            got_i, got_d, _ = srv.run(tiny.queries[:nq], off, ids, in_flight=in_flight)
            assert np.array_equal(got_i, to_np(ref_i)) and np.array_equal(got_d, to_np(ref_d))
    finally:
        assert srv.end() == (2 * nq, 1)


@pytest.mark.parametrize("waves,n_workers", [(8, 1023), (4, 1023), (1, 1023), (8, 256), (8, 223)])
def test_other_work_runs_beside_a_session_of_many_workers(vf, waves, n_workers):
    """float32 workers take a compute unit's whole register file: however many are asked for, a copy that is a kernel (up to
    16 KiB) still runs beside them, with up to 223 larger kernels too, and the session goes on.  (What cannot run waits for the
    idle bound, and the session is over.)"""
    import torch
    w = make_workload("c2", n=12_000, nq=64, n_labels=20, n_clusters=16, T=800, graph_degree=16)
    s = w.spec
    X = torch.from_numpy(w.vectors).cuda()
    ix = vf.build_index(X, w.label_offsets, w.label_ids, s.n_labels, s.T, s.graph_degree)
    words = torch.ones(512 * 1024, device="cuda")
    words.add_(1)
    torch.cuda.synchronize()
    srv = vf.Server(ix, 10, n_workers=n_workers, waves_per_worker=waves, ring_slots=64, idle_polls=200_000, itopk=32, width=1, iters=6, n_seeds=64)
    try:
        first = srv.run(w.queries, w.qlabel_offsets, w.qlabel_ids, in_flight=64)
        for i in range(3):
            if n_workers == 223:
                words.add_(1)
            assert (words[:3072].cpu() == (3 + i if n_workers == 223 else 2)).all()
        again = srv.run(w.queries, w.qlabel_offsets, w.qlabel_ids, in_flight=64)
        assert np.array_equal(first[0], again[0]) and np.array_equal(first[1], again[1])
    finally:
        done, why = srv.end()
    assert (done, why) == (2 * s.nq, 1)


def test_a_small_idle_bound_outlasts_short_pauses(vf, tiny):
    """A counted poll takes a few microseconds from the first one on: 64 of them are longer than pauses of 130 us between jobs,
    also where polls are quick at first."""
    import torch
    s = tiny.spec
    X = torch.from_numpy(tiny.vectors).cuda()
    ix = vf.build_index(X, tiny.label_offsets, tiny.label_ids, s.n_labels, s.T, s.graph_degree)
    lasted = False
    for _ in range(20):   # (the host may be held up for longer than that)
        srv = vf.Server(ix, 10, itopk=32, width=1, iters=4, n_seeds=64, n_workers=8, ring_slots=64, idle_polls=64)
        try:
            for _ in range(12):
                srv.submit(tiny.queries[0], [int(tiny.qlabel_ids[0])])
                t0 = time.perf_counter()
                while time.perf_counter() - t0 < 130e-6:
                    pass
            lasted = True
        except vf.VecflowError as e:
            assert "ended" in str(e)
        srv.end()
        if lasted:
            break
    assert lasted


def test_jobs_submitted_before_the_idle_bound_are_finished(vf, tiny):
    """One worker with a queue of jobs, which take longer together than the dispatcher's own last wait: all are done."""
    import torch
    s = tiny.spec
    X = torch.from_numpy(tiny.vectors).cuda()
    ix = vf.build_index(X, tiny.label_offsets, tiny.label_ids, s.n_labels, s.T, s.graph_degree)
    nq, off = 256, tiny.qlabel_offsets
    for _ in range(20):   # (the host may be held up for longer than the idle bound while it submits)
        srv = vf.Server(ix, 10, itopk=64, width=1, iters=30, n_seeds=64, n_workers=1, waves_per_worker=1, ring_slots=nq, idle_polls=300)
        jobs = []
        try:
            for j in range(nq):
                jobs.append(srv.submit(tiny.queries[j], tiny.qlabel_ids[off[j]:off[j + 1]].tolist()))
        except vf.VecflowError as e:
            assert "ended" in str(e)
        got = _wait(srv, jobs)
        done, why = srv.end()
        assert len(got) == done == len(jobs) and why in (1, 3)
        if done == nq:
            return
    pytest.fail("the host was held up every time")
