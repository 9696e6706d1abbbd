"""Dimensions without a seed kernel of their own score their seeds densely, through the next larger instantiation, or leave
them to the beam kernel, by the number of seeds and queries: which of the two on either side of each line, and the same
results."""
import numpy as np
import pytest

from oracle import OracleIndex
from tests.gpu_util import assert_exact, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,dim,n_seeds,nq,dense", [
    ("float32", 4, 256, 3, True), ("float32", 36, 191, 65, False), ("float32", 36, 192, 65, True),
    ("float32", 100, 0, 1, False), ("float32", 100, 383, 70, False), ("float32", 100, 384, 70, True),
    ("float32", 132, 1023, 1, False), ("float32", 132, 1024, 128, True), ("float32", 248, 1024, 129, False),
    ("float32", 200, 4096, 600, False), ("uint8", 80, 32, 64, False), ("uint8", 80, 300, 64, True),
    ("uint8", 272, 383, 5, False), ("uint8", 272, 777, 5, True), ("uint8", 992, 512, 64, True),
    ("uint8", 992, 512, 1100, False), ("float32", 128, 32, 1, True), ("float32", 36, 1024, 9, True), ("float32", 100, 2048, 9, True),
    ("float32", 200, 8192, 70, True), ("uint8", 528, 2048, 9, True)])
@pytest.mark.parametrize("pairs", [False, True])
def test_dense_or_gathered(dtype, dim, n_seeds, nq, dense, pairs):
    import torch
    from paper_2506_00812_amd import binding as vf
    rng = np.random.default_rng(dim + n_seeds)
    n, R = 1500, 8
    x = rng.normal(size=(12, dim))[rng.integers(0, 12, n)] * (30 if dtype == "uint8" else 2) + rng.normal(size=(n, dim)) * (12 if dtype == "uint8" else 1)
    x = np.rint(x + 128).clip(0, 255).astype(np.uint8) if dtype == "uint8" else x.astype(np.float32)
    carry = rng.random((n, 3)) < [0.9, 0.5, 0.3]
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    asked = [[0], [1], [2], [0, 1], [0]]
    if pairs:   # queries with a predicate for the most part: more seeds
        asked = [[0, 1], [1, 2], [2], [0, 2], [0, 1]]
        own = dim * (1 if dtype == "uint8" else 4) // 16 in (8, 12, 16, 24, 32)
        chunks = dim * (1 if dtype == "uint8" else 4) // 16
        dense = own or max(n_seeds, 64) >= (1024 if chunks <= 16 else 2048 if chunks <= 32 or dtype == "uint8" else 8192)
    asked = [asked[j % 5] for j in range(nq)]
    qoff = np.concatenate([[0], np.cumsum([len(a) for a in asked])]).astype(np.int64)
    qids = np.array([l for a in asked for l in a], dtype=np.int32)
    q = x[rng.integers(0, n, nq)]
    if dtype == "float32":
        q = (q + 0.5 * rng.normal(size=q.shape)).astype(np.float32)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, 3, 50, R)
    ixo = OracleIndex(x, off, ids, 3, 50, R)
    # float32 dim 128 has a matrix-core form for lists of up to 48 entries; beyond them it scores with the ordered distance
    params = dict(itopk=64, width=1, iters=6, n_seeds=n_seeds)
    ix.profile_enable(True)
    gi, gd = vf.search(ix, torch.from_numpy(np.ascontiguousarray(q)).cuda(), qoff, qids, 10, **params)
    assert (ix.profile_read()["n_seed_tiles"] > 0) == dense
    oi, od = ixo.search(q, qoff, qids, 10, **params)
    assert_exact(to_np(gi), to_np(gd), oi, od, "seeds")
