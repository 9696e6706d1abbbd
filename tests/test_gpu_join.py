"""The join kernel (self-joins of the index build) at the edges of its tiles: lists around whole groups of 32 entries and
whole tiles of 32 and 128 rows, dimensions around the contraction steps it is compiled for, candidate counts up to its 64."""
import numpy as np
import pytest

from oracle import OracleIndex

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,dim,R", [("float32", 4, 5), ("float32", 36, 32), ("float32", 100, 24), ("float32", 128, 48),
                                         ("float32", 132, 32), ("float32", 248, 32), ("uint8", 16, 7), ("uint8", 80, 64),
                                         ("uint8", 208, 32), ("uint8", 528, 16), ("uint8", 992, 32)])
def test_graph_rows_at_tile_edges(dtype, dim, R):
    import torch
    from paper_2506_00812_amd import binding as vf
    rng = np.random.default_rng(dim + R)
    sizes = [R + 1, max(R + 1, 95), 96, 97, 127, 128, 129, 257, 900]
    n = 1000
    centres = rng.normal(size=(8, dim)) * (30 if dtype == "uint8" else 2) + (128 if dtype == "uint8" else 0)
    x = centres[rng.integers(0, 8, n)] + rng.normal(size=(n, dim)) * (12 if dtype == "uint8" else 1)
    x = np.rint(x).clip(0, 255).astype(np.uint8) if dtype == "uint8" else x.astype(np.float32)
    x[10:14] = x[5]                                     # equal distances are ordered by id
    labels = [[] for _ in range(n)]
    for l, size in enumerate(sizes):
        for i in np.sort(rng.permutation(n)[:size]):
            labels[i].append(l)
    off = np.concatenate([[0], np.cumsum([len(v) for v in labels])]).astype(np.int64)
    ids = np.array([l for v in labels for l in v], dtype=np.int32)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, len(sizes), R + 1, R)
    want = OracleIndex(x, off, ids, len(sizes), R + 1, R).G_HS
    got = ix.export("G_HS").reshape(-1, R)
    bad = np.flatnonzero((got != want).any(axis=1))
    assert len(bad) == 0, f"{len(bad)} of {len(got)} rows differ, first {bad[:3]}: {got[bad[0]]} {want[bad[0]]}"


@pytest.mark.parametrize("dtype,dim,k", [("float32", 100, 10), ("float32", 128, 1), ("float32", 96, 48), ("float32", 40, 49),
                                         ("float32", 244, 64), ("uint8", 128, 10), ("uint8", 48, 64), ("uint8", 400, 7)])
def test_exact_search_at_tile_edges(dtype, dim, k):
    """Ground truth over graph lists: one, 128, 129 and 300 queries of a label, lists of several segments, AND queries, k up
    to the largest for which spare candidates are kept and beyond it."""
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_close_with_ties, assert_exact, to_np
    rng = np.random.default_rng(dim + k)
    n, n_labels = 9000, 8
    centres = rng.normal(size=(16, dim)) * (30 if dtype == "uint8" else 2) + (128 if dtype == "uint8" else 0)

    def points(count):
        x = centres[rng.integers(0, 16, count)] + rng.normal(size=(count, dim)) * (12 if dtype == "uint8" else 1)
        return np.rint(x).clip(0, 255).astype(np.uint8) if dtype == "uint8" else x.astype(np.float32)

    x = points(n)
    x[100:130] = x[7]                                   # equal distances are ordered by id
    share = np.array([0.95, 0.5, 0.3, 0.1, 0.05, 0.012, 0.004, 0.0])
    carry = rng.random((n, n_labels)) < share
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    asked = [[0]] * 300 + [[1]] * 129 + [[2]] * 128 + [[3]] + [[4]] * 5 + [[5]] * 3 + [[6]] * 2 + [[7]] + [[0, 1]] * 40 + \
            [[1, 2, 3]] * 20 + [[0, 5]] * 10 + [[0, 7]]
    order = rng.permutation(len(asked))
    asked = [asked[i] for i in order]
    qoff = np.concatenate([[0], np.cumsum([len(a) for a in asked])]).astype(np.int64)
    qids = np.array([l for a in asked for l in a], dtype=np.int32)
    q = points(len(asked))
    q[3], q[4] = x[7], x[8]
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, n_labels, 200, 16)
    ixo = OracleIndex(x, off, ids, n_labels, 200, 16, lazy_graph=True)
    for count in (len(asked), 1):
        gi, gd = vf.search_exact(ix, torch.from_numpy(q[:count]).cuda(), qoff[:count + 1], qids[:qoff[count]], k)
        oi, od = ixo.search(q[:count], qoff[:count + 1], qids[:qoff[count]], k, force_scan=True)
        if dtype == "uint8":
            assert_exact(to_np(gi), to_np(gd), oi, od, "exact")
        else:
            assert_close_with_ties(to_np(gi), to_np(gd), oi, od, 1e-4, "exact")


def _shifted(dim, shift, spread, n=6000, nq=200):
    rng = np.random.default_rng(dim)
    centres = rng.normal(size=(12, dim)) * spread + shift
    x = (centres[rng.integers(0, 12, n)] + rng.normal(size=(n, dim))).astype(np.float32)
    q = (centres[rng.integers(0, 12, nq)] + rng.normal(size=(nq, dim))).astype(np.float32)
    carry = rng.random((n, 2)) < [0.99, 0.5]
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    return x, q, off, np.nonzero(carry)[1].astype(np.int32), carry


def _truth(x, q, member, k):
    """The k nearest members of every query in 64 bits."""
    at = np.flatnonzero(member)
    v, q = x[at].astype(np.float64), q.astype(np.float64)
    d = ((q[:, None, :] - v[None, :, :]) ** 2).sum(2) if len(at) * q.size < 1 << 28 else \
        np.stack([((q[j] - v) ** 2).sum(1) for j in range(len(q))])
    order = np.argsort(d, axis=1, kind="stable")[:, :k]
    return at[order], np.take_along_axis(d, order, 1)


@pytest.mark.parametrize("dim", [40, 100, 128, 132, 248])
def test_tables_far_from_the_origin(dim):
    """A table and its queries shifted by 30 (noise 1, clusters of 500): every row and result has its proof, and is right."""
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_close_with_ties, to_np
    x, q, off, ids, carry = _shifted(dim, 30.0, 2.0)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, 2, 100, 16)
    rows = ix.export("G_HS").reshape(-1, 16)
    member = np.flatnonzero(carry[:, 0])
    local, _ = _truth(x, x[member[:40]], carry[:, 0], 17)
    for j in range(40):   # (the row's own vertex is the nearest of its list)
        assert set(member[rows[j]]) == set(local[j, 1:])
    ix.profile_enable(True)
    for label in (0, 1):
        qoff, qids = np.arange(len(q) + 1, dtype=np.int64), np.full(len(q), label, dtype=np.int32)
        gi, gd = vf.search_exact(ix, torch.from_numpy(q).cuda(), qoff, qids, 10)
        wi, wd = _truth(x, q, carry[:, label], 10)
        assert_close_with_ties(to_np(gi), to_np(gd), wi, wd.astype(np.float32), 1e-5, "exact")
    assert ix.profile_read()["scan_fallbacks"] == 0


def test_proofs_of_the_ground_truth_are_not_weakened():
    """Clusters so far apart that some proofs fail: as many of them with "seed_slack" below 1 as at 1, the same results."""
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_close_with_ties, to_np
    x, q, off, ids, carry = _shifted(128, 0.0, 150.0)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, 2, 100, 16)
    qoff, qids = np.arange(len(q) + 1, dtype=np.int64), np.zeros(len(q), dtype=np.int32)
    failed = []
    for slack in (1.0, 0.001):
        ix.tune("seed_slack", slack)
        ix.profile_enable(True)
        gi, gd = vf.search_exact(ix, torch.from_numpy(q).cuda(), qoff, qids, 10)
        wi, wd = _truth(x, q, carry[:, 0], 10)
        assert_close_with_ties(to_np(gi), to_np(gd), wi, wd.astype(np.float32), 1e-5, "exact")
        failed.append(ix.profile_read()["scan_fallbacks"])
    assert failed[0] == failed[1] > 0


@pytest.mark.parametrize("dim,k,sizes,nq", [(128, 10, [9000, 4000, 700, 130], 300), (100, 48, [9000, 2500, 400], 60), (4, 1, [3000, 129], 5000),
                                            (96, 25, [6000, 65, 64, 33], 400), (248, 7, [1030, 200], 41)])
def test_ground_truth_without_proofs(dim, k, sizes, nq):
    """A bound that no result meets sends every query of a float32 graph list (and of a scan list, in batches that filter) to
    the ordered scan: one query or many of a list, AND queries, several segments; the results keep their bits.  Queries with
    NaN, infinities and overflowing norms go there by themselves."""
    import torch
    from paper_2506_00812_amd import binding as vf
    rng = np.random.default_rng(dim + k)
    n, T = max(sizes) + 50, 300
    x = ((rng.normal(size=(16, dim)) * 2)[rng.integers(0, 16, n)] + rng.normal(size=(n, dim))).astype(np.float32)
    carry = np.zeros((n, len(sizes)), dtype=bool)
    for l, size in enumerate(sizes):
        carry[rng.permutation(n)[:size], l] = True
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    asked = [[l] for l in range(len(sizes))] + [[0, 1], [0, len(sizes) - 1]]
    asked += [sorted(set(rng.integers(0, len(sizes), rng.integers(1, 3)).tolist())) for _ in range(nq - len(asked))]
    qoff = np.concatenate([[0], np.cumsum([len(a) for a in asked])]).astype(np.int64)
    qids = np.array([l for a in asked for l in a], dtype=np.int32)
    q = x[rng.integers(0, n, nq)] + 0.5 * rng.normal(size=(nq, dim)).astype(np.float32)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, len(sizes), T, 8)
    ix.profile_enable(True)

    def search(q):
        out = vf.search_exact(ix, torch.from_numpy(np.ascontiguousarray(q)).cuda(), qoff, qids, k)
        return [t.cpu().numpy() for t in out], ix.profile_read()["scan_fallbacks"]

    (ids0, d0), _ = search(q)
    graph = np.array([min(int(carry[:, l].sum()) for l in a) >= T for a in asked])
    ix.tune("seed_slack", 1e6)
    ix.profile_enable(True)
    (ids1, d1), failed = search(q)
    # (a query with fewer members than are kept needs no proof)
    enough = np.array([int(carry[:, a].all(1).sum()) >= min(64, k + 22) for a in asked])
    assert failed >= (graph & enough).sum() > 0
    assert np.array_equal(ids0[graph], ids1[graph]) and np.array_equal(d0[graph].view(np.uint32), d1[graph].view(np.uint32))
    assert np.array_equal(ids0, ids1) and np.allclose(d0, d1, rtol=1e-5)
    ix.tune("seed_slack", 1.0)
    odd = {0: np.nan, 1: np.inf, 4: -np.inf, 5: 3e19}
    q2 = q.copy()
    for j, v in odd.items():
        if j < nq:
            q2[j, dim // 2] = v
    (ids2, d2), failed = search(q2)
    rest = [j for j in range(nq) if j not in odd]
    assert np.array_equal(ids2[rest], ids0[rest])
    for j, v in odd.items():
        if graph[j]:   # all distances are the same: the lowest ids
            want = np.flatnonzero(carry[:, asked[j]].all(1))[:k]
            assert np.array_equal(ids2[j][:len(want)], want) and (ids2[j][len(want):] == -1).all()
            assert np.isnan(d2[j][:len(want)]).all() if np.isnan(v) else np.isinf(d2[j]).all()


@pytest.mark.parametrize("spread,dim,R", [(4, 32, 16), (12, 64, 16), (12, 96, 32), (0, 80, 16), (12, 100, 32), (12, 128, 48), (60, 236, 32)])
def test_rows_that_binary16_does_not_prove(spread, dim, R):
    """Clusters so far apart that the rounding of the operands to binary16 hides the order of a row's neighbours: those rows are
    joined again on split operands, in segments of their lists, a few of them, most, or all."""
    import torch
    from tests.gpu_util import assert_close_with_ties, to_np
    from paper_2506_00812_amd import binding as vf
    rng = np.random.default_rng(spread + dim)
    n, sizes = 5000, [4800, 2000, 700]
    centres = rng.normal(size=(12, dim)) * spread
    x = (centres[rng.integers(0, 12, n)] + rng.normal(size=(n, dim))).astype(np.float32)
    if spread == 0:                                     # equal points: no operands prove anything
        x = np.repeat(x[:50], 100, axis=0)
    labels = [[] for _ in range(n)]
    for l, size in enumerate(sizes):
        for i in np.sort(rng.permutation(n)[:size]):
            labels[i].append(l)
    off = np.concatenate([[0], np.cumsum([len(v) for v in labels])]).astype(np.int64)
    ids = np.array([l for v in labels for l in v], dtype=np.int32)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, len(sizes), 600, R)
    want = OracleIndex(x, off, ids, len(sizes), 600, R)
    assert np.array_equal(ix.export("G_HS").reshape(-1, R), want.G_HS)
    q = (centres[rng.integers(0, 12, 260)] + rng.normal(size=(260, dim))).astype(np.float32)
    qoff, qids = np.arange(261), (np.arange(260) % 3).astype(np.int32)
    for k in (1, 25):
        gi, gd = vf.search_exact(ix, torch.from_numpy(q).cuda(), qoff, qids, k)
        wi, wd = want.search(q, qoff, qids, k, force_scan=True)
        assert_close_with_ties(to_np(gi), to_np(gd), wi, wd, 1e-4, f"k {k}")


def test_long_lists_are_tried_before_they_are_joined():
    """A list long enough that a few of its rows decide which operands the join takes, near clusters and far ones: the rows are
    those of the scan kernels."""
    import torch
    from paper_2506_00812_amd import binding as vf
    n, dim, R = 66_000, 32, 16
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    off, ids = np.arange(n + 1, dtype=np.int64), np.zeros(n, dtype=np.int32)
    for spread in (2.0, 40.0):
        centres = torch.randn((500, dim), generator=g, device="cuda") * spread
        x = centres[torch.randint(0, 500, (n,), generator=g, device="cuda")] + torch.randn((n, dim), generator=g, device="cuda")
        got = vf.build_index(x, off, ids, 1, 1000, R).export("G_HS")
        vf.tune_defaults("build16", 0)
        try:
            want = vf.build_index(x, off, ids, 1, 1000, R).export("G_HS")
        finally:
            vf.tune_defaults("build16", 1)
        assert np.array_equal(got, want), f"clusters {spread} apart"


def test_rows_of_several_lists_are_tried():
    """The same with three lists whose pairs together make a look worth its time; clusters so far apart that half the rows or
    all have no proof, where everything is joined again, and near ones."""
    import torch
    from paper_2506_00812_amd import binding as vf
    n, dim, R, sizes = 40_000, 36, 24, [30_007, 20_000, 16_001]
    rng = np.random.default_rng(8)
    carry = np.zeros((n, 3), dtype=bool)
    for l, size in enumerate(sizes):
        carry[rng.permutation(n)[:size], l] = True
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    for spread in (1.5, 12.0, 50.0):
        centres = rng.normal(size=(300, dim)) * spread
        x = torch.from_numpy((centres[rng.integers(0, 300, n)] + rng.normal(size=(n, dim))).astype(np.float32)).cuda()
        got = vf.build_index(x, off, ids, 3, 1000, R).export("G_HS")
        vf.tune_defaults("build16", 0)
        try:
            want = vf.build_index(x, off, ids, 3, 1000, R).export("G_HS")
        finally:
            vf.tune_defaults("build16", 1)
        assert np.array_equal(got, want), f"clusters {spread} apart"


def _table(dtype, dim, n, sizes, spread, seed):
    """Clustered points with some equal ones, posting lists of the given sizes, and a function that draws more points."""
    rng = np.random.default_rng(seed)
    centres = rng.normal(size=(16, dim)) * (30 if dtype == "uint8" else spread) + (128 if dtype == "uint8" else 0)

    def points(count):
        x = centres[rng.integers(0, 16, count)] + rng.normal(size=(count, dim)) * (12 if dtype == "uint8" else 1)
        return np.rint(x).clip(0, 255).astype(np.uint8) if dtype == "uint8" else x.astype(np.float32)

    x = points(n)
    x[100:130] = x[7]
    carry = np.zeros((n, len(sizes)), dtype=bool)
    for l, size in enumerate(sizes):
        carry[rng.permutation(n)[:size], l] = True
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    return x, off, np.nonzero(carry)[1].astype(np.int32), points


def _check_exact(ix, ixo, q, asked, k, what):
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_close_with_ties, assert_exact, to_np
    qoff = np.concatenate([[0], np.cumsum([len(a) for a in asked])]).astype(np.int64)
    qids = np.array([l for a in asked for l in a], dtype=np.int32)
    gi, gd = vf.search_exact(ix, torch.from_numpy(q).cuda(), qoff, qids, k)
    oi, od = ixo.search(q, qoff, qids, k, force_scan=True)
    (assert_exact if q.dtype == np.uint8 else lambda *a: assert_close_with_ties(*a[:4], 1e-4, a[4]))(to_np(gi), to_np(gd), oi, od, what)


@pytest.mark.parametrize("dtype,dim,spread", [("float32", 100, 2), ("float32", 96, 60), ("float32", 128, 60), ("float32", 132, 2), ("float32", 244, 60),
                                              ("uint8", 256, 0), ("uint8", 272, 0), ("uint8", 528, 0), ("uint8", 976, 0), ("uint8", 992, 0)])
def test_few_queries_of_long_lists(dtype, dim, spread):
    """Lone queries and a few: lists of one wave and, from 16 steps of the contraction on, of four; operands in registers and,
    of the last of 32 steps, in LDS; segments whose first thresholds come from a few groups, from many and from none."""
    import torch
    from paper_2506_00812_amd import binding as vf
    sizes = [9000, 1030, 530, 500]
    x, off, ids, points = _table(dtype, dim, 9500, sizes, spread, dim)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, len(sizes), 200, 16)
    ixo = OracleIndex(x, off, ids, len(sizes), 200, 16, lazy_graph=True)
    q = points(12)
    q[1] = x[7]
    for k, counts in ((1, (1, 6)), (5, (1, 5, 12)), (24, (1, 2, 6))):
        for nq in counts:
            _check_exact(ix, ixo, q[:nq], [[0]] * nq, k, f"{nq} queries, k {k}")
        _check_exact(ix, ixo, q, [[0], [1], [2], [3], [0, 1], [2, 3], [1, 2]] + [[0]] * 3 + [[1]] * 2, k, f"several lists, k {k}")


@pytest.mark.parametrize("dtype,dim,k", [("float32", 64, 48), ("float32", 128, 10), ("uint8", 128, 64)])
def test_queries_around_the_rows_of_a_small_tile(dtype, dim, k):
    """Lists with a few queries are cut into tiles of 8, 16 or 32 rows: numbers of queries around them, ties, AND queries."""
    import torch
    from paper_2506_00812_amd import binding as vf
    sizes = [9000, 4500, 700]
    x, off, ids, points = _table(dtype, dim, 9500, sizes, 2, dim + k)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, len(sizes), 200, 16)
    ixo = OracleIndex(x, off, ids, len(sizes), 200, 16, lazy_graph=True)
    q = points(100)
    q[1] = x[7]
    for nq in (7, 8, 9, 17, 31, 33, 100):
        _check_exact(ix, ixo, q[:nq], [[0]] * nq, k, f"{nq} queries")
    _check_exact(ix, ixo, q, [[0]] * 41 + [[1]] * 23 + [[2]] * 9 + [[0, 1]] * 16 + [[0, 1, 2]] * 11, k, "several lists")


@pytest.mark.parametrize("dim,R,spread", [(128, 16, 3), (128, 16, 4), (64, 16, 4), (128, 8, 5), (128, 32, 2), (64, 32, 12)])
def test_ground_truth_that_binary16_would_not_prove(dim, R, spread):
    """Tables whose rows binary16 operands prove, but not the queries, or not those for many results: the index knows it from its
    build, and the first call finds its proofs as a later one does.  A call whose queries go without proofs changes nothing."""
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_close_with_ties, to_np
    rng = np.random.default_rng(dim + R)
    n, nq = 20_000, 1000
    centres = rng.normal(size=(40, dim)) * spread
    x = (centres[rng.integers(0, 40, n)] + rng.normal(size=(n, dim))).astype(np.float32)
    q = (centres[rng.integers(0, 40, nq)] + rng.normal(size=(nq, dim))).astype(np.float32)
    off, ids = np.arange(n + 1, dtype=np.int64), np.zeros(n, dtype=np.int32)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, 1, 1000, R)
    qoff, qids, Q = np.arange(nq + 1, dtype=np.int64), np.zeros(nq, dtype=np.int32), torch.from_numpy(q).cuda()

    def unproven(count, k):
        ix.profile_enable(True)
        gi, gd = vf.search_exact(ix, Q[:count], qoff[:count + 1], qids[:count], k)
        wi, wd = _truth(x, q[:40], np.ones(n, dtype=bool), k)
        m = min(count, 40)
        assert_close_with_ties(to_np(gi)[:m], to_np(gd)[:m], wi[:m], wd[:m].astype(np.float32), 1e-5, f"k {k}")
        return ix.profile_read()["scan_fallbacks"]

    def few(counts):   # (1 in 64 rows may be without a proof, and as many queries)
        return all(c <= n_c // 32 for c, n_c in counts)

    def all_counts():
        return [(unproven(count, k), count) for k in (10, 26, 42, 48) for count in (40, nq)]

    first = all_counts()
    assert few(first), first
    ix.tune("seed_slack", 1e6)
    assert unproven(nq, 10) == nq
    ix.tune("seed_slack", 1.0)
    assert all_counts() == first


@pytest.mark.parametrize("dtype,dim,k,spread", [("float32", 36, 10, 2), ("float32", 128, 10, 2), ("float32", 128, 10, 60), ("float32", 96, 42, 2),
                                                ("float32", 132, 7, 60), ("float32", 248, 10, 2), ("uint8", 128, 10, 0), ("uint8", 192, 64, 0),
                                                ("uint8", 272, 5, 0), ("uint8", 976, 10, 0)])
def test_many_queries_of_each_list(dtype, dim, k, spread):
    """Ground truth with 257 queries per list and more: lists of several segments, last tiles of 1, 44 and 129 rows (from 16 steps on
    in workgroups with waves without rows), filtered queries between others, ties; operands of one part and of two, in one LDS
    buffer, in two and in registers."""
    import torch
    from paper_2506_00812_amd import binding as vf
    sizes = [9000, 2500, 700]
    x, off, ids, points = _table(dtype, dim, 9500, sizes, spread, dim + k)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, len(sizes), 200, 16)
    ixo = OracleIndex(x, off, ids, len(sizes), 200, 16, lazy_graph=True)
    rng = np.random.default_rng(k)
    for counts in ((385, 300, 257), (513, 257, 0)):
        asked = [[0]] * counts[0] + [[1]] * counts[1] + [[2]] * counts[2]
        pairs = [[0, 1]] * 40 + [[1, 2]] * 30 + [[0, 2]] * 20 + [[0, 1, 2]] * 10
        for a in (asked, asked + pairs):
            a = [a[i] for i in rng.permutation(len(a))]
            q = points(len(a))
            q[3], q[4] = x[7], x[8]
            _check_exact(ix, ixo, q, a, k, f"{counts} queries")


@pytest.mark.parametrize("dim,k", [(128, 10), (36, 16), (96, 1), (248, 5)])
def test_queries_beyond_binary16(dim, k):
    """Finite queries around the norm from which ground truth takes no binary16 operands (31,622 in the operands' unit), around the
    largest binary16 number (65,504) and far above it: results as from the ordered scan alone, in lists of any length."""
    import torch
    from paper_2506_00812_amd import binding as vf
    sizes = [9000, 700, 60, 39, 38, 33, 32, 31, 22]
    x, off, ids, points = _table("float32", dim, 9500, sizes, 2, dim)
    unit = 2.0 ** (6 - np.frexp(np.linalg.norm(x - x.mean(0), axis=1).max())[1])
    targets = np.array([3e3, 2.9e4, 3.1e4, 3.16e4, 3.17e4, 3.3e4, 6.4e4, 6.55e4, 6.6e4, 1e5, 1e6, 1e9]) / unit
    q = []
    for j, t in enumerate(targets):
        for sign in (1, -1):
            one, all_ = points(1)[0], points(1)[0]
            one[j % dim] += sign * t
            all_ += sign * t / np.sqrt(dim)
            q += [one, all_]
    q = np.array(q + list(points(8)), dtype=np.float32)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, len(sizes), 20, 16)
    for label in range(len(sizes)):
        asked = np.full(len(q), label, dtype=np.int32)
        out = []
        for slack in (1.0, 1e6):
            ix.tune("seed_slack", slack)
            gi, gd = vf.search_exact(ix, torch.from_numpy(q).cuda(), np.arange(len(q) + 1), asked, k)
            out.append((gi.cpu().numpy(), gd.cpu().numpy()))
        (gi, gd), (wi, wd) = out
        bad = np.flatnonzero((gi != wi).any(1) | (gd.view(np.uint32) != wd.view(np.uint32)).any(1))
        assert len(bad) == 0, f"list of {sizes[label]}: queries {bad}: {gi[bad[0]]} {wi[bad[0]]}"
