"""The bound of approximate seeds for tables whose norms are near the ends of the admitted range (squared norms of 1e-24 to 1e30),
with the query's own rounding to binary16 as the term that matters: the query is orthogonal to the seeds' direction, and its
rounding errors all point along it, so the approximations prefer the wrong half of the seeds by more than the rest of the bound."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [128, 96, 100, 36])
@pytest.mark.parametrize("exponent", [-40, -20, 0, 30, 40])
def test_rounding_of_the_query(dim, exponent):
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact, to_np
    rng = np.random.default_rng(dim)
    n, nq, half = 700, 600, dim // 2
    q1 = np.concatenate([np.full(half, 1 + 0.99 * 2.0 ** -11), np.full(half, -(1 + 1.01 * 2.0 ** -11))])
    x = np.rint((-0.75 * q1 + 0.1 * rng.normal(size=(n, dim))) * 64) / 64        # every component is a binary16 number
    place = rng.permutation(n)
    x[place[:40]] = 1.0
    x[place[:40], half:half + 1] -= 2.0 ** -7                                    # nearer to the query than ...
    x[place[40:80]] = -1.0                                                       # ... these; after rounding it is further
    x, q = (x * 2.0 ** exponent).astype(np.float32), (np.tile(q1, (nq, 1)) * 2.0 ** exponent).astype(np.float32)
    d = ((q[0].astype(np.float64) - x.astype(np.float64)) ** 2).sum(1)
    assert np.array_equal(np.argsort(d, kind="stable")[:40], np.sort(place[:40]))
    off, ids = np.arange(n + 1, dtype=np.int64), np.zeros(n, dtype=np.int32)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, 1, 200, 8)
    Q, qoff, qids = torch.from_numpy(q).cuda(), np.arange(nq + 1), np.zeros(nq, dtype=np.int32)
    params = dict(itopk=32, width=1, iters=0, n_seeds=n)
    ix.profile_enable(True)
    got = [to_np(t) for t in vf.search(ix, Q, qoff, qids, 10, **params)]
    pf = ix.profile_read()
    ix.profile_enable(False)
    session = vf.Server(ix, 10, n_workers=16, **params)
    try:
        ids_s, d_s, _ = session.run(q[:40], qoff[:41], qids[:40], in_flight=16)
    finally:
        session.end()
    ix.tune("seed_exact", 1)
    want = [to_np(t) for t in vf.search(ix, Q, qoff, qids, 10, **params)]
    assert np.array_equal(want[0][0], np.sort(place[:40])[:10])
    assert_exact(*got, *want, "batch")
    assert_exact(ids_s, d_s, want[0][:40], want[1][:40], "session")
    assert pf["seeds_on_matrix_cores"] == 2 and pf["seed_fallbacks"] == 0
