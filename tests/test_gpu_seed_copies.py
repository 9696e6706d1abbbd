"""The copies of the seeds that calls make and keep: searches with new seed counts beside a serving session, and more seed counts than
an index keeps copies of."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _table(dtype, dim, n=12_000, nq=300, seed=0):
    rng = np.random.default_rng(dim + seed)
    x = rng.normal(size=(20, dim))[rng.integers(0, 20, n)] * 2 + rng.normal(size=(n, dim))
    q = x[rng.integers(0, n, nq)] + 0.4 * rng.normal(size=(nq, dim))
    x, q = ((np.rint(a * 25 + 128).clip(0, 255).astype(np.uint8) if dtype == "uint8" else a.astype(np.float32)) for a in (x, q))
    carry = rng.random((n, 3)) < [0.9, 0.5, 0.1]
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    return x, off, np.nonzero(carry)[1].astype(np.int32), q, np.arange(nq + 1), rng.integers(0, 3, nq).astype(np.int32)


@pytest.mark.parametrize("dtype,dim", [("float32", 100), ("float32", 200), ("float32", 36), ("uint8", 112), ("uint8", 400)])
def test_new_seed_counts_beside_a_session(dtype, dim):
    """Dimensions without a kernel instantiation of their own: a call with a new seed count waits for no session, whether it makes a
    copy of the seeds or there are as many as are kept.  (A wait for the device is one for the session's idle bound, and the session
    is over.)"""
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact, to_np
    x, off, ids, q, qoff, qids = _table(dtype, dim)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, 3, 300, 16)
    Q = torch.from_numpy(q).cuda()
    params = dict(itopk=32, width=1, iters=5)
    outs = [(torch.empty((len(q), 10), dtype=torch.int64, device="cuda"), torch.empty((len(q), 10), device="cuda")) for _ in range(6)]
    ix.profile_enable(True)
    vf.search(ix, Q, qoff, qids, 10, n_seeds=3000, out_ids=outs[0][0], out_dists=outs[0][1], **params)      # the workspace is at its size
    ix.profile_read()
    torch.cuda.synchronize()
    counts = (2500, 1200, 800, 500, 300, 200)     # the last three: beyond the copies that are kept
    srv = vf.Server(ix, 10, n_workers=32, ring_slots=64, idle_polls=200_000, n_seeds=1000, **params)
    try:
        first = srv.run(q, qoff, qids, in_flight=32)
        on = []
        for n_seeds, (oi, od) in zip(counts, outs):
            vf.search(ix, Q, qoff, qids, 10, n_seeds=n_seeds, out_ids=oi, out_dists=od, **params)
            on.append(ix.profile_read()["seeds_on_matrix_cores"])
        again = srv.run(q, qoff, qids, in_flight=32)
    finally:
        done, why = srv.end()
    assert (done, why) == (2 * len(q), 1)
    assert on == [2 if dtype == "float32" else 1] * 3 + [0] * 3
    assert_exact(first[0], first[1], again[0], again[1], "session")
    ix.tune("seed_exact", 1)
    for n_seeds, (oi, od) in zip(counts, outs):
        want = vf.search(ix, Q, qoff, qids, 10, n_seeds=n_seeds, **params)
        assert_exact(to_np(oi), to_np(od), to_np(want[0]), to_np(want[1]), f"{n_seeds} seeds")


def _stingy(vf, device):
    """An allocator that refuses the sizes in al.refuse (bytes, or "large": above 100,000), and counts what it has refused."""
    al = vf.TorchAllocator(device)
    inner, al.refuse, al.refused = al._alloc_cb, set(), 0

    def alloc(nbytes, ctx):
        if nbytes > 100_000 if al.refuse == "large" else nbytes in al.refuse:
            al.refused += 1
            return None
        return inner(nbytes, ctx)
    al.cb = vf.ALLOC_FN(alloc)
    al.struct = vf.VfAllocator(al.cb, al._free_cb, None)
    return al


def _build_with(vf, al, X, *args):
    real = vf.TorchAllocator
    vf.TorchAllocator = lambda device: al
    try:
        return vf.build_index(X, *args)
    finally:
        vf.TorchAllocator = real


@pytest.mark.parametrize("dtype,dim", [("float32", 100), ("float32", 128), ("uint8", 112), ("uint8", 192)])
def test_no_memory_for_a_copy(dtype, dim):
    """An allocator that gives nothing large any more, or not the binary16 copy: the search and the session do without, with the same results."""
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact, to_np
    x, off, ids, q, qoff, qids = _table(dtype, dim, nq=600)
    X, Q = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda()
    n_seeds, workers = 1500, 16
    params = dict(itopk=32, width=1, iters=5, n_seeds=n_seeds)
    sizes = [int(s) for s in np.bincount(ids, minlength=3)]
    groups = sum((min(n_seeds, s) + 31) // 32 for s in sizes)
    up = lambda b: (b + 255) & ~255
    group_bytes = 2 * ((dim * (1 if dtype == "uint8" else 4) + 31) // 32) * 512
    stride = (max(min(n_seeds, s) for s in sizes) + 31) & ~31
    rows = workers * (stride + ((stride // 32 + 63) & ~63)) * 4
    al = _stingy(vf, X.device)
    ix = _build_with(vf, al, X, off, ids, 3, 300, 16)
    ix.tune("seed_exact", 1)
    want = [to_np(t) for t in vf.search(ix, Q, qoff, qids, 10, **params)]      # (and the workspace is at its size)
    ix.tune("seed_exact", 0)
    al.refuse = "large"
    for _ in range(2):
        got = vf.search(ix, Q, qoff, qids, 10, **params)
        assert_exact(to_np(got[0]), to_np(got[1]), *want, "batch without a copy")
    assert al.refused > 0
    for refuse in ({up(groups * group_bytes // 2)}, {up(rows)}, {up(groups * group_bytes)}):
        al.refuse, al.refused = refuse, 0
        srv = vf.Server(ix, 10, n_workers=workers, ring_slots=64, **params)
        try:
            ids_s, d_s, _ = srv.run(q, qoff, qids, in_flight=32)
        finally:
            assert srv.end() == (len(q), 1)
        assert al.refused == (1 if dtype == "float32" or refuse == {up(groups * group_bytes)} else 0)
        assert_exact(ids_s, d_s, *want, f"session without a block of {refuse} bytes")
    al.refuse = set()
    ix2 = _build_with(vf, al, X, off, ids, 3, 300, 16)
    al.refuse, al.refused = {up(groups * group_bytes // 2)}, 0                 # (float32: the binary16 form alone)
    got = vf.search(ix2, Q, qoff, qids, 10, **params)
    assert al.refused == (1 if dtype == "float32" else 0)
    assert_exact(to_np(got[0]), to_np(got[1]), *want, "batch without the binary16 copy")


@pytest.mark.parametrize("dtype,dim,itopk,n_seeds,labels", [
    ("float32", 100, 64, 300, [[0], [1]]), ("uint8", 400, 64, 300, [[0], [1]]),      # lists of 64 entries, few seeds: gathered
    ("float32", 100, 64, 1000, [[0, 1]]), ("float32", 128, 64, 1000, [[0, 1]]),      # ... with predicates: by the ordered distance
    ("float32", 100, 32, 1000, [[2]]), ("uint8", 112, 32, 1000, [[2]])])             # lists that are scanned
def test_no_copy_for_calls_that_do_not_use_it(dtype, dim, itopk, n_seeds, labels):
    """A call that scores no seeds from a copy makes none: as many blocks of memory as with copies switched off."""
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact, to_np
    x, off, ids, q, _, _ = _table(dtype, dim)
    asked = [labels[j % len(labels)] for j in range(len(q))]
    qoff = np.concatenate([[0], np.cumsum([len(a) for a in asked])]).astype(np.int64)
    qids = np.array([l for a in asked for l in a], dtype=np.int32)
    X, Q = torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda()
    found = []
    for cache in (1, 0):
        ix = vf.build_index(X, off, ids, 3, 2000, 16)        # (the third list is scanned)
        ix.tune("seed_cache", cache)
        before = ix.allocator.n_alloc
        out = vf.search(ix, Q, qoff, qids, 10, itopk=itopk, width=1, iters=5, n_seeds=n_seeds)
        found.append(([to_np(t) for t in out], ix.allocator.n_alloc - before))
    assert found[0][1] == found[1][1]
    assert_exact(*found[0][0], *found[1][0], "without copies")


@pytest.mark.parametrize("dtype,dim", [("float32", 100), ("float32", 128), ("float32", 248), ("uint8", 128), ("uint8", 528)])
def test_more_seeds_than_any_list_has(dtype, dim):
    """Seed counts up to the largest number there is mean every entry of a list."""
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact, to_np
    x, off, ids, q, qoff, qids = _table(dtype, dim, n=5000)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, 3, 300, 16)
    Q = torch.from_numpy(q).cuda()
    for nq in (1, 300):
        want = None
        for n_seeds in (5000, (1 << 23) + 1, (1 << 30) + 5, 2 ** 31 - 32, 2 ** 31 - 31, 2 ** 31 - 1):
            got = [to_np(t) for t in vf.search(ix, Q[:nq], qoff[:nq + 1], qids[:nq], 10, itopk=32, width=1, iters=3, n_seeds=n_seeds)]
            want = want or got
            assert_exact(*got, *want, f"{n_seeds} seeds")
        exact = vf.search_exact(ix, Q[:nq], qoff[:nq + 1], qids[:nq], 10)
        assert np.array_equal(to_np(exact[0]), want[0])
