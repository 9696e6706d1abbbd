"""Ground truth of float32 tables in which one vector occurs many times: the copies are at one distance and equal to the rounded value
that a row's first threshold is taken from, so all of them pass it or none.  Queries on the copied vector's ray beyond it and on the
other side (where q.x - |x|^2 / 2 is not exact), zero rows among isotropic ones, lists of one segment and of several, predicates."""
import numpy as np
import pytest

from oracle import OracleIndex

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,k", [(128, 1), (128, 10), (128, 42), (64, 25), (36, 10), (96, 42), (132, 10)])
@pytest.mark.parametrize("zero", [False, True])
def test_copies_of_one_vector(dim, k, zero):
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_close_with_ties, assert_exact, to_np
    rng = np.random.default_rng(dim + k)
    n, sizes = 9500, [9000, 3000, 1030, 600]
    carry = np.zeros((n, len(sizes)), dtype=bool)
    for l, size in enumerate(sizes):
        carry[rng.permutation(n)[:size], l] = True
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    base = rng.normal(size=(n, dim))
    one = np.zeros(dim) if zero else rng.normal(size=dim)
    copies = rng.permutation(n)[:n // 10]
    asked = [[l] for l in range(len(sizes))] * 12 + [[0, 1], [0, 2], [1, 3], [0, 1, 2]]
    qoff = np.concatenate([[0], np.cumsum([len(a) for a in asked])]).astype(np.int64)
    qids = np.array([l for a in asked for l in a], dtype=np.int32)
    for scale in np.arange(1.0, 2.0, 0.1):
        x = base * (scale if zero else 1.0)
        x[copies] = one * scale
        x = x.astype(np.float32)
        if zero:      # any direction, short enough that the zero rows are the nearest
            q = rng.normal(size=(len(asked), dim)) * 0.3
        else:
            q = one * scale * np.repeat([1.3, 2.0, 2.7, -1.0, 0.9, 1.01], len(asked) // 6 + 1)[:len(asked), None] + 0.01 * rng.normal(size=(len(asked), dim))
        q = q.astype(np.float32)
        ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, len(sizes), 500, 16)
        got = [to_np(t) for t in vf.search_exact(ix, torch.from_numpy(q).cuda(), qoff, qids, k)]
        want = OracleIndex(x, off, ids, len(sizes), 500, 16, lazy_graph=True).search(q, qoff, qids, k, force_scan=True)
        assert_close_with_ties(*got, *want, 1e-4, f"scale {scale:.1f}")
        ix.tune("seed_slack", 1e6)      # no proofs: every list by the definition
        plain = [to_np(t) for t in vf.search_exact(ix, torch.from_numpy(q).cuda(), qoff, qids, k)]
        assert_exact(*got, *plain, f"scale {scale:.1f}, by the definition")
