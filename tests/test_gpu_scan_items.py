"""How many work items a batch's scans are cut into: what one list gets does not depend on the other lists of the batch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _index(dtype, dim, sizes, T, n=5000):
    import torch
    from paper_2506_00812_amd import binding as vf
    rng = np.random.default_rng(dim)
    x = rng.normal(size=(n, dim)) * 20 + 128
    x = np.rint(x).clip(0, 255).astype(np.uint8) if dtype == "uint8" else (x - 128).astype(np.float32)
    carry = np.zeros((n, len(sizes)), dtype=bool)
    for l, size in enumerate(sizes):
        carry[rng.permutation(n)[:size], l] = True
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    X = torch.from_numpy(x).cuda()
    ix = vf.build_index(X, off, ids, len(sizes), T, 8)
    ix.profile_enable(True)
    return ix, X


def _asked(labels):
    return np.arange(len(labels) + 1, dtype=np.int64), np.array(labels, dtype=np.int32)


@pytest.mark.parametrize("dtype,dim,k", [("float32", 40, 64), ("float32", 128, 50)])
def test_exact_graph_lists_beside_scan_lists(dtype, dim, k):
    """k of more than 48: graph lists go through the scan kernels, list by list."""
    from paper_2506_00812_amd import binding as vf
    ix, X = _index(dtype, dim, [4000, 3000, 500, 70], T=1000)

    def items(labels):
        vf.search_exact(ix, X[:len(labels)], *_asked(labels), k)
        return ix.profile_read()["n_scan_items"]

    graph = items([0] * 9 + [1])
    assert graph == 8 + 6          # 125 and 94 groups, 16 to a segment
    for scans in ([2], [3], [2] * 20, [2, 3] * 10):
        assert items([0] * 9 + [1] + scans) == graph + items(scans)
