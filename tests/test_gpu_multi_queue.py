"""Calls queued one after the other without waiting, with routing blobs that are read in place from host memory or uploaded,
by their size: the staging buffers, the blobs and the workspace's buffers are used again by the calls that follow.  The
parents of vf_search_multi's sub-searches travel with the blob."""
import numpy as np
import pytest

from paper_2506_00812_amd.workloads import make_workload
from tests.gpu_util import to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("zero_copy_bytes", [0, 8192, 32768])
def test_queued_calls(zero_copy_bytes):
    import torch
    from paper_2506_00812_amd import binding as vf
    w = make_workload("c2", n=40_000, nq=3000, n_labels=80, n_clusters=64, T=1200, graph_degree=16, seed=5)
    X = torch.from_numpy(w.vectors).cuda()
    ix = vf.build_index(X, w.label_offsets, w.label_ids, 80, 1200, 16)
    ix.tune("zero_copy_bytes", zero_copy_bytes)
    rng = np.random.default_rng(1)
    params = dict(itopk=32, width=1, iters=6, n_seeds=512)
    calls = []
    for i, nq in enumerate([1, 2900, 3, 700, 300, 301, 299, 2500, 17, 400, 64, 1, 1500, 250]):
        asked = [rng.permutation(80)[:rng.integers(1, 4)] for _ in range(nq)]
        qoff = np.concatenate([[0], np.cumsum([len(a) for a in asked])]).astype(np.int64)
        Q = torch.from_numpy(w.queries[rng.integers(0, len(w.queries), nq)]).cuda()
        mode = [vf.OR, vf.AND_PARALLEL, vf.OR, vf.OR | vf.MULTI_EXACT][i % 4]
        calls.append((Q, qoff, np.concatenate(asked).astype(np.int32), mode))

    def run(c):
        return vf.search_multi(ix, c[0], c[1], c[2], c[3], 10, **params)

    want = []
    for c in calls:
        got = run(c)
        torch.cuda.synchronize()
        want.append([to_np(t) for t in got])
    for _ in range(3):
        got = [run(c) for c in calls]
        torch.cuda.synchronize()
        for g, v in zip(got, want):
            assert np.array_equal(to_np(g[0]), v[0]) and np.array_equal(to_np(g[1]), v[1])


def test_queued_searches_around_the_size_that_is_read_in_place():
    """The scan path on its side stream, batches around the 32 KiB of routing that are no longer uploaded."""
    import torch
    from paper_2506_00812_amd import binding as vf
    w = make_workload("c2", n=40_000, nq=3000, n_labels=80, n_clusters=64, T=1200, graph_degree=16, seed=6)
    ix = vf.build_index(torch.from_numpy(w.vectors).cuda(), w.label_offsets, w.label_ids, 80, 1200, 16)
    rng = np.random.default_rng(2)
    params = dict(itopk=32, width=1, iters=6, n_seeds=512)
    calls = []
    for nq in list(range(200, 2600, 150)) + [800, 2500, 900, 850, 3000, 1000]:
        asked = [rng.permutation(80)[:rng.integers(1, 3)] for _ in range(nq)]
        qoff = np.concatenate([[0], np.cumsum([len(a) for a in asked])]).astype(np.int64)
        calls.append((torch.from_numpy(w.queries[rng.integers(0, len(w.queries), nq)]).cuda(), qoff, np.concatenate(asked).astype(np.int32)))

    def run():
        out = [vf.search(ix, *c, 10, **params) for c in calls]
        torch.cuda.synchronize()
        return [(to_np(i), to_np(d)) for i, d in out]

    got = [run() for _ in range(3)]
    ix.tune("zero_copy_bytes", 0)
    ix.tune("overlap", 0)
    want = run()
    for g in got:
        for a, b in zip(g, want):
            assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
