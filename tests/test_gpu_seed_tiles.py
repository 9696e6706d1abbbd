"""Seed tiles of 64 queries and the binary16 copy of the seeds: tiles of one query, one set and a row more or less, lists that end
inside a group, tables of very large and very small numbers, and queries that binary16 cannot hold: the ordered distances' results."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,dim,scale", [("uint8", 192, 1), ("uint8", 112, 1), ("float32", 128, 1), ("float32", 96, 1e-6), ("float32", 96, 1e9),
                                             ("float32", 60, 37.0)])
def test_tiles_of_64(dtype, dim, scale):
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact, to_np
    rng = np.random.default_rng(dim)
    counts = [1, 31, 32, 33, 63, 64, 65, 97, 128, 129, 400]       # queries of each label: 1,043, with 8,200 seeds asked for
    sizes = [8300, 8193, 8192, 1025, 1023, 513, 511, 300, 8160, 8161, 900]
    n = 9000
    x = rng.normal(size=(20, dim))[rng.integers(0, 20, n)] * 2 + rng.normal(size=(n, dim))
    q = x[rng.integers(0, n, sum(counts))] + 0.3 * rng.normal(size=(sum(counts), dim))
    if dtype == "uint8":
        x, q = (np.rint(a * 25 + 128).clip(0, 255).astype(np.uint8) for a in (x, q))
    else:
        x, q = ((a * scale).astype(np.float32) for a in (x, q))
        q[5] *= 1e4                                                # beyond the range that the table's scale leaves
    carry = np.zeros((n, len(sizes)), dtype=bool)
    for l, size in enumerate(sizes):
        carry[rng.permutation(n)[:size], l] = True
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    qids = rng.permutation(np.repeat(np.arange(len(counts), dtype=np.int32), counts))
    qoff = np.arange(len(qids) + 1)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, len(sizes), 200, 16)
    Q = torch.from_numpy(q).cuda()
    params = dict(itopk=32, width=1, iters=3, n_seeds=8200)
    ix.profile_enable(True)
    got = vf.search(ix, Q, qoff, qids, 10, **params)
    pf = ix.profile_read()
    ix.profile_enable(False)
    assert pf["seeds_on_matrix_cores"] == (2 if dtype == "float32" else 1)
    assert pf["seed_fallbacks"] == (1 if dtype == "float32" else 0)
    ix.tune("seed_exact", 1)
    want = vf.search(ix, Q, qoff, qids, 10, **params)
    assert_exact(to_np(got[0]), to_np(got[1]), to_np(want[0]), to_np(want[1]), "tiles of 64")
