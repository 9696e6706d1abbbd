"""Seeds on the matrix cores for dimensions without an instantiation of their own (fewer contraction steps than the kernel has,
an odd number of chunks, a chunk half empty, the largest that is taken and the first that is not) and for lists of up to 64
entries: the results of the ordered distances, one, four and sixteen groups of seeds per wave, with and without block minima
and predicates."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,dim,on_matrix_cores", [
    ("float32", 4, 2), ("float32", 36, 2), ("float32", 100, 2), ("float32", 132, 2), ("float32", 248, 2), ("uint8", 16, 1),
    ("uint8", 112, 1), ("uint8", 240, 1), ("uint8", 512, 1), ("uint8", 528, 0)])
@pytest.mark.parametrize("nq,n_seeds,itopk,pairs", [(1, 777, 32, 0.0), (300, 195, 16, 0.0), (1700, 1100, 48, 0.0), (1500, 3300, 32, 0.0),
                                                    (900, 1300, 32, 0.7), (5000, 1000, 64, 0.0)])
def test_same_results(dtype, dim, on_matrix_cores, nq, n_seeds, itopk, pairs):
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact, to_np
    rng = np.random.default_rng(dim + nq)
    n, n_labels = 9000, 3
    centres = rng.normal(size=(30, dim)) * (30 if dtype == "uint8" else 2) + (128 if dtype == "uint8" else 0)

    def points(count):
        x = centres[rng.integers(0, 30, count)] + rng.normal(size=(count, dim)) * (12 if dtype == "uint8" else 1)
        return np.rint(x).clip(0, 255).astype(np.uint8) if dtype == "uint8" else x.astype(np.float32)

    carry = rng.random((n, n_labels)) < np.array([0.95, 0.5, 0.1])   # the last list is shorter than some seed counts
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    two = rng.random(nq) < pairs
    qoff = np.concatenate([[0], np.cumsum(1 + two)]).astype(np.int64)
    first = rng.integers(0, n_labels, nq)
    qids = np.empty(qoff[-1], dtype=np.int32)
    qids[qoff[:-1]] = first
    qids[qoff[:-1][two] + 1] = (first[two] + 1) % n_labels
    ix = vf.build_index(torch.from_numpy(points(n)).cuda(), off, ids, n_labels, 500, 16)
    Q = torch.from_numpy(points(nq)).cuda()
    params = dict(itopk=itopk, width=1, iters=4, n_seeds=n_seeds)
    ix.profile_enable(True)
    got = vf.search(ix, Q, qoff, qids, 10, **params)
    assert ix.profile_read()["seeds_on_matrix_cores"] == on_matrix_cores
    ix.profile_enable(False)
    ix.tune("seed_exact", 1)     # every seed's ordered distance
    want = vf.search(ix, Q, qoff, qids, 10, **params)
    assert_exact(to_np(got[0]), to_np(got[1]), to_np(want[0]), to_np(want[1]), "seeds")


@pytest.mark.parametrize("dim", [96, 100, 128])
@pytest.mark.parametrize("pairs", [False, True])
def test_lists_of_64_entries(dim, pairs):
    """float32 lists beyond 48 entries: on the matrix cores without predicates, by the ordered distance with them; a bound that never
    holds makes every wave score its seeds itself."""
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact, to_np
    rng = np.random.default_rng(dim)
    n, nq = 6000, 700
    x = (rng.normal(size=(20, dim))[rng.integers(0, 20, n)] * 2 + rng.normal(size=(n, dim))).astype(np.float32)
    q = (x[rng.integers(0, n, nq)] + 0.5 * rng.normal(size=(nq, dim))).astype(np.float32)
    carry = rng.random((n, 2)) < [0.9, 0.6]
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    qoff = np.arange(nq + 1) * (2 if pairs else 1)
    qids = np.tile(np.array([0, 1], dtype=np.int32), nq)[:qoff[-1]]
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, 2, 300, 24)
    Q = torch.from_numpy(q).cuda()
    found = []
    for knob, value in ((None, 0), ("seed_slack", 1e30), ("seed_exact", 1)):
        if knob:
            ix.tune(knob, value)
        for n_seeds, iters in ((700, 5), (2600, 0)):
            ix.profile_enable(True)
            got = vf.search(ix, Q, qoff, qids, 25, itopk=64, width=2, iters=iters, n_seeds=n_seeds)
            pf = ix.profile_read()
            ix.profile_enable(False)
            found.append([to_np(t) for t in got])
            on = knob != "seed_exact" and not pairs
            assert (pf["seeds_on_matrix_cores"] > 0) == on
            assert pf["seed_fallbacks"] == (nq if knob == "seed_slack" and on else 0)
    for a, b in zip(found[:4], found[4:] + found[4:]):
        assert_exact(*a, *b, "lists of 64")
