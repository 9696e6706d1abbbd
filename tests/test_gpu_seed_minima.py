"""Seed selection through the minima of 32-seed blocks (large batches with many seeds): the same results as the route that
scores and offers every seed, on ordinary data, on data full of equal distances (more ties than the selection has room
for), for lists shorter than the seed count, and with part of the batch carrying a predicate."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,dim,noise,itopk,n_seeds,pairs", [
    ("uint8", 192, 12, 32, 4096, 0.0), ("uint8", 128, 12, 64, 6161, 0.3), ("uint8", 192, 0, 32, 4096, 0.0),
    ("uint8", 128, 0.4, 32, 33000, 0.2), ("float32", 128, 1, 16, 6144, 0.0), ("float32", 96, 1, 10, 4100, 0.0),
    ("float32", 128, 0, 10, 6144, 0.0)])
def test_block_minima_change_nothing(dtype, dim, noise, itopk, n_seeds, pairs):
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact, to_np
    rng = np.random.default_rng(dim + n_seeds)
    n, nq, n_labels, T = 30_000, 4500, 5, 1500
    centres = rng.normal(size=(40, dim)) * (30 if dtype == "uint8" else 2) + (128 if dtype == "uint8" else 0)

    def points(count):
        x = centres[rng.integers(0, 40, count)] + rng.normal(size=(count, dim)) * noise
        return np.rint(x).clip(0, 255).astype(np.uint8) if dtype == "uint8" else x.astype(np.float32)

    x, q = points(n), points(nq)
    carry = rng.random((n, n_labels)) < np.array([0.95, 0.6, 0.3, 0.1, 0.06])
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    two = rng.random(nq) < pairs
    qoff = np.concatenate([[0], np.cumsum(1 + two)]).astype(np.int64)
    first = rng.integers(0, n_labels, nq)
    qids = np.empty(qoff[-1], dtype=np.int32)
    qids[qoff[:-1]] = first
    qids[qoff[:-1][two] + 1] = (first[two] + 1) % n_labels
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, n_labels, T, 16)
    Q = torch.from_numpy(q).cuda()
    params = dict(itopk=itopk, width=1, iters=4, n_seeds=n_seeds)
    got = vf.search(ix, Q, qoff, qids, 10, **params)
    ix.tune("seed_exact", 1)     # every seed's ordered distance, no matrix cores, no minima
    want = vf.search(ix, Q, qoff, qids, 10, **params)
    assert_exact(to_np(got[0]), to_np(got[1]), to_np(want[0]), to_np(want[1]), "block minima")


@pytest.mark.parametrize("nq", [1, 33, 500, 1500])
@pytest.mark.parametrize("dtype,dim,noise", [("uint8", 192, 12), ("float32", 128, 1), ("float32", 96, 0)])
def test_block_minima_of_small_batches(dtype, dim, noise, nq):
    """One, four and sixteen groups of seeds per wave, searches by the latency and the throughput kernel; a seed count that ends
    within a block."""
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact, to_np
    rng = np.random.default_rng(nq + dim)
    n = 20_000
    centres = rng.normal(size=(40, dim)) * (30 if dtype == "uint8" else 2) + (128 if dtype == "uint8" else 0)

    def points(count):
        x = centres[rng.integers(0, 40, count)] + rng.normal(size=(count, dim)) * noise
        return np.rint(x).clip(0, 255).astype(np.uint8) if dtype == "uint8" else x.astype(np.float32)

    carry = rng.random((n, 3)) < np.array([0.95, 0.5, 0.2])
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    Q, qoff, qids = torch.from_numpy(points(nq)).cuda(), np.arange(nq + 1), rng.integers(0, 3, nq).astype(np.int32)
    ix = vf.build_index(torch.from_numpy(points(n)).cuda(), off, ids, 3, 1500, 16)
    params = dict(itopk=16, width=2, iters=4, n_seeds=5003)
    got = vf.search(ix, Q, qoff, qids, 10, **params)
    ix.tune("seed_exact", 1)
    want = vf.search(ix, Q, qoff, qids, 10, **params)
    assert_exact(to_np(got[0]), to_np(got[1]), to_np(want[0]), to_np(want[1]), "block minima")
