"""Candidate distances of the beam search for vectors of every number of 16-byte chunks that its kernels tell apart (one, a team's
eight and one more, sixteen, thirty-two and one more, rows that end inside a step), in the instantiations for few and for many
queries, against the oracle; seed counts that divide the list, do not, or cover it."""
import numpy as np
import pytest

from oracle import OracleIndex

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,dim", [("uint8", 16), ("uint8", 48), ("uint8", 128), ("uint8", 144), ("uint8", 272), ("uint8", 528),
                                       ("float32", 4), ("float32", 32), ("float32", 36), ("float32", 68), ("float32", 128), ("float32", 132)])
def test_candidate_distances(dtype, dim):
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact, to_np
    rng = np.random.default_rng(dim)
    n, nq = 4000, 2300
    x = rng.normal(size=(10, dim))[rng.integers(0, 10, n)] * 2 + rng.normal(size=(n, dim))
    q = x[rng.integers(0, n, nq)] + 0.4 * rng.normal(size=(nq, dim))
    x, q = ((np.rint(a * 25 + 128).clip(0, 255).astype(np.uint8) if dtype == "uint8" else a.astype(np.float32)) for a in (x, q))
    carry = rng.random((n, 2)) < [0.9, 0.3]
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, 2, 300, 20)
    ixo = OracleIndex(x, off, ids, 2, 300, 20)
    for count, two in ((3, False), (1300, False), (nq, False), (300, True), (1300, True)):
        per = 2 if two else 1
        qoff = np.arange(count + 1) * per
        qids = (np.tile([0, 1], count) if two else rng.integers(0, 2, count)).astype(np.int32)
        Q = torch.from_numpy(q[:count]).cuda()
        for params in (dict(itopk=32, width=2, iters=6, n_seeds=100), dict(itopk=16, width=1, iters=9, n_seeds=5000)):
            ids_g, d_g = vf.search(ix, Q, qoff, qids, 10, **params)
            ids_o, d_o = ixo.search(q[:count], qoff, qids, 10, **params)
            assert_exact(to_np(ids_g), to_np(d_g), ids_o, d_o.astype(np.float32), f"{count} {two} {params}")
