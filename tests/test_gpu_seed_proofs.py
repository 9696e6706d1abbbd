"""Where approximate float32 seeds give way to ordered distances: tables far from the origin, whose norms hide the distances from the
proofs, and proofs that fail."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _index(vf, dim, shift, n=8000, nq=2100):
    import torch
    rng = np.random.default_rng(dim)
    x = rng.normal(size=(20, dim))[rng.integers(0, 20, n)] * 2 + rng.normal(size=(n, dim)) + shift
    q = (x[rng.integers(0, n, nq)] + 0.4 * rng.normal(size=(nq, dim))).astype(np.float32)
    carry = rng.random((n, 2)) < [0.9, 0.5]
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ix = vf.build_index(torch.from_numpy(x.astype(np.float32)).cuda(), off, np.nonzero(carry)[1].astype(np.int32), 2, 300, 16)
    return ix, torch.from_numpy(q).cuda(), np.arange(nq + 1), rng.integers(0, 2, nq).astype(np.int32)


def _search(vf, ix, Q, qoff, qids, **params):
    from tests.gpu_util import to_np
    ix.profile_enable(True)
    out = [to_np(t) for t in vf.search(ix, Q, qoff, qids, 10, width=1, iters=4, **params)]
    pf = ix.profile_read()
    ix.profile_enable(False)
    return out, pf


@pytest.mark.parametrize("dim,itopk,near", [(100, 32, 2), (200, 32, 2), (100, 64, 2), (128, 64, 2)])
def test_tables_far_from_the_origin(dim, itopk, near):
    """Dimensions without a kernel instantiation of their own and lists of more than 48 entries: on the matrix cores near the origin, by
    the ordered distance far from it, with the same results; sessions too."""
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact, to_np
    for shift, on in ((0.0, near), (1.0, near), (40.0, 0), (3000.0, 0)):
        ix, Q, qoff, qids = _index(vf, dim, shift)
        params = dict(itopk=itopk, n_seeds=1000)
        for nq in (600, 2100):
            got, pf = _search(vf, ix, Q[:nq], qoff[:nq + 1], qids[:nq], **params)
            assert pf["seeds_on_matrix_cores"] == on and pf["seed_fallbacks"] == 0, (shift, nq)
        q = to_np(Q)
        session = vf.Server(ix, 10, n_workers=16, width=1, iters=4, **params)
        try:
            ids_s, d_s, _ = session.run(q, qoff, qids, in_flight=32)
        finally:
            session.end()
            del session      # (an index that is freed waits for the device)
        ix.tune("seed_exact", 1)
        want, _ = _search(vf, ix, Q, qoff, qids, **params)
        assert_exact(*got, *want, f"shift {shift}")
        assert_exact(ids_s, d_s, *want, f"shift {shift}, session")


@pytest.mark.parametrize("dim,itopk", [(100, 32), (128, 64)])
def test_failing_proofs_are_noticed_early(dim, itopk):
    """Proofs that fail: calls that have ordered distances to go back to do so after the first few thousand queries, and wait for
    nothing; others of the same index go on."""
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact
    ix, Q, qoff, qids = _index(vf, dim, 0.0)
    params = dict(itopk=itopk, n_seeds=700)
    want, pf = _search(vf, ix, Q, qoff, qids, **params)
    assert pf["seeds_on_matrix_cores"] == 2 and pf["seed_fallbacks"] == 0
    live = ix.allocator.live_bytes()
    ix.tune("seed_slack", 1e30)      # no bound holds
    seen = []
    for _ in range(4):
        got, pf = _search(vf, ix, Q, qoff, qids, **params)
        assert_exact(*got, *want, "failed proofs")
        seen.append((pf["seeds_on_matrix_cores"], pf["seed_fallbacks"]))
    assert seen == [(2, len(Q))] + [(0, 0)] * 3
    assert ix.allocator.live_bytes() >= live          # the copies stay: nothing has waited for the device
    if dim == 128:
        ix.tune("seed_slack", 1.0)
        _, pf = _search(vf, ix, Q, qoff, qids, itopk=32, n_seeds=700)
        assert pf["seeds_on_matrix_cores"] == 2


@pytest.mark.parametrize("dim,nq", [(160, 1), (160, 300), (232, 40)])
def test_predicates_that_few_seeds_pass(dim, nq):
    """Wide vectors: seeds are scored on the matrix cores where enough of them pass, and gathered where few do."""
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact
    rng = np.random.default_rng(dim)
    n = 10_000
    x = rng.normal(size=(20, dim))[rng.integers(0, 20, n)] * 2 + rng.normal(size=(n, dim))
    Q = torch.from_numpy((x[rng.integers(0, n, nq)] + 0.4 * rng.normal(size=(nq, dim))).astype(np.float32)).cuda()
    carry = np.zeros((n, 3), dtype=bool)
    for l, size in enumerate((600, 6000, 1000)):     # of the first list's seeds 360 carry the second label, 60 the third
        carry[rng.permutation(n)[:size], l] = True
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ix = vf.build_index(torch.from_numpy(x.astype(np.float32)).cuda(), off, np.nonzero(carry)[1].astype(np.int32), 3, 300, 16)
    qoff = np.arange(nq + 1) * 2
    for other, on in ((1, 2), (2, 0)):
        qids = np.tile([0, other], nq).astype(np.int32)
        got, pf = _search(vf, ix, Q, qoff, qids, itopk=32, n_seeds=2000)
        assert pf["seeds_on_matrix_cores"] == on
        ix.tune("seed_exact", 1)
        want, _ = _search(vf, ix, Q, qoff, qids, itopk=32, n_seeds=2000)
        ix.tune("seed_exact", 0)
        assert_exact(*got, *want, f"partner {other}")
