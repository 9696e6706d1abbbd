"""Serving sessions whose workers filter the seeds from their binary16 copy: dimensions with and without an instantiation and the
largest there is, seed counts that end inside a group or leave waves without a share, one, four and eight waves, predicates in
between, and bounds that never hold: the batched search's results."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [4, 36, 96, 100, 128, 248])
@pytest.mark.parametrize("waves,n_seeds,slack", [(8, 193, 1.0), (8, 5000, 1.0), (4, 1500, 1.0), (1, 777, 1.0), (8, 1500, 1e30)])
def test_same_results(dim, waves, n_seeds, slack):
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact, to_np
    rng = np.random.default_rng(dim + n_seeds)
    n, nq = 6000, 250
    x = (rng.normal(size=(20, dim))[rng.integers(0, 20, n)] * 2 + rng.normal(size=(n, dim))).astype(np.float32)
    q = (x[rng.integers(0, n, nq)] + 0.4 * rng.normal(size=(nq, dim))).astype(np.float32)
    q[7] *= 1e5                                                         # beyond what binary16 holds at the table's scale
    carry = rng.random((n, 3)) < [0.9, 0.35, 0.04]
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, 3, 400, 24)
    ix.tune("seed_slack", slack)
    two = rng.random(nq) < 0.2
    qoff = np.concatenate([[0], np.cumsum(1 + two)]).astype(np.int64)
    qids = np.empty(qoff[-1], dtype=np.int32)
    first = rng.integers(0, 3, nq)
    qids[qoff[:-1]] = first
    qids[qoff[:-1][two] + 1] = (first[two] + 1) % 3
    params = dict(itopk=32, width=2, iters=5, n_seeds=n_seeds)
    with_session = vf.Server(ix, 10, waves_per_worker=waves, **params)
    ids_s, d_s, _ = with_session.run(q, qoff, qids, in_flight=33)
    assert with_session.end()[0] == nq
    ids_b, d_b = vf.search(ix, torch.from_numpy(q).cuda(), qoff, qids, 10, **params)
    assert_exact(ids_s, d_s, to_np(ids_b), to_np(d_b), "session")
