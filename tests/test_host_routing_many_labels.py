"""CPU tests of how a batch is grouped by label where few and where many labels are asked for (the order of the labels comes from
sorting them or from a bitmap of all labels), with queries of one, two equal, two and three labels and some without an answer."""
import numpy as np
import pytest

from paper_2506_00812_amd import binding as vf


@pytest.mark.parametrize("n_labels,nq", [(70, 3000), (65, 64), (4096, 63), (4096, 700), (5000, 20000), (100_000, 300)])
def test_groups(n_labels, nq):
    rng = np.random.default_rng(n_labels + nq)
    T = 200
    S = rng.integers(1, 400, n_labels).astype(np.int32)
    S[rng.integers(0, n_labels, max(1, n_labels // 50))] = 0
    counts = rng.choice([1, 2, 3], nq, p=[0.4, 0.5, 0.1])
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    ids = rng.integers(0, n_labels, off[-1]).astype(np.int32)
    ids[off[:-1][::7] + (counts[::7] == 2)] = ids[off[:-1][::7]]        # some twice the same label
    r = vf.debug_route(S, T, off, ids)
    searched = np.empty(nq, dtype=np.int64)
    for j in range(nq):
        labs = np.unique(ids[off[j]:off[j + 1]])
        searched[j] = -1 if (S[labs] == 0).any() else min(labs, key=lambda l: (S[l], l))
        assert r["n_others"][j] == (0 if searched[j] < 0 else len(labs) - 1)
    assert np.array_equal(r["searched"], searched)
    graph = (searched >= 0) & (S[searched] >= T)
    assert np.array_equal(r["method"], np.where(searched < 0, 0, np.where(graph, 2, 1)))
    by_label = np.argsort(searched, kind="stable")
    assert np.array_equal(r["graph_queries"], by_label[graph[by_label]])
    scan = (searched >= 0) & ~graph
    assert np.array_equal(r["scan_rows"], by_label[scan[by_label]])
