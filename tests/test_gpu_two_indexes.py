"""Calls on two indexes in turn on one stream, nothing waited for and results dropped at once: a workspace buffer that a
later call allocates may be a block that queued work of the caller's stream still writes."""
import numpy as np
import pytest

from paper_2506_00812_amd.workloads import make_workload
from tests.gpu_util import to_np

pytestmark = pytest.mark.gpu


def test_dropped_results_of_another_index():
    import torch
    from paper_2506_00812_amd import binding as vf
    w = [make_workload("c2", n=60_000, nq=6000, n_labels=100, n_clusters=64, T=1500, graph_degree=16, seed=s) for s in (1, 2)]
    params = dict(itopk=32, width=2, iters=12, n_seeds=1024)
    X = [torch.from_numpy(v.vectors).cuda() for v in w]
    Q = [torch.from_numpy(v.queries).cuda() for v in w]

    def build(i):
        return vf.build_index(X[i], w[i].label_offsets, w[i].label_ids, 100, 1500, 16)

    def search(ix, i):
        return vf.search(ix, Q[i], w[i].qlabel_offsets, w[i].qlabel_ids, 10, **params)

    want = []
    for i in (0, 1):
        ix = build(i)
        got = search(ix, i)
        torch.cuda.synchronize()
        want.append([to_np(t) for t in got])
        del ix, got
    for _ in range(3):
        ixs = [build(0), build(1)]
        torch.cuda.synchronize()
        for i in (0, 1, 1):       # results dropped
            search(ixs[i], i)
        last = [search(ixs[0], 0), search(ixs[1], 1)]
        torch.cuda.synchronize()
        for i in (0, 1):
            assert np.array_equal(to_np(last[i][0]), want[i][0]) and np.array_equal(to_np(last[i][1]), want[i][1])
