"""AND queries on the filtering scan (float32, batches of more than 256 scan queries): its predicate masks cover windows of
768 entries, so lists and segments around and beyond that, with partners that are graph lists, scan lists, both, or empty."""
import numpy as np
import pytest

from oracle import OracleIndex
from tests.gpu_util import assert_close_with_ties, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,seg_groups,slots", [(128, 24, 1), (96, 24, 2), (128, 23, 1), (96, 49, 1), (128, 64, 2), (96, 1, 1)])
def test_and_masks_at_window_edges(dim, seg_groups, slots):
    import torch
    from paper_2506_00812_amd import binding as vf
    rng = np.random.default_rng(dim + seg_groups)
    n, k, T = 6000, 10, 2500
    x = (rng.normal(size=(24, dim)) * 2)[rng.integers(0, 24, n)] + rng.normal(size=(n, dim))
    x = x.astype(np.float32)
    sizes = [4500, 3000, 2400, 1537, 1536, 769, 768, 767, 33, 32, 31, 1, 0]
    carry = np.zeros((n, len(sizes)), dtype=bool)
    for l, size in enumerate(sizes):
        carry[rng.permutation(n)[:size], l] = True
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    asked = []
    for j in range(500):
        m = [1, 2, 2, 2, 3, 4][j % 6]
        asked.append(sorted(set(rng.integers(0 if j % 2 else 2, len(sizes) if j % 50 == 0 else 12, m).tolist())))
    qoff = np.concatenate([[0], np.cumsum([len(a) for a in asked])]).astype(np.int64)
    qids = np.array([l for a in asked for l in a], dtype=np.int32)
    q = (x[rng.integers(0, n, 500)] + 0.5 * rng.normal(size=(500, dim))).astype(np.float32)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, len(sizes), T, 16)
    ix.tune("scan_bf16_seg_groups", seg_groups)
    ix.tune("scan_bf16_slots", slots)
    ixo = OracleIndex(x, off, ids, len(sizes), T, 16, lazy_graph=True)
    params = dict(itopk=32, width=1, iters=8, n_seeds=256)
    ix.profile_enable(True)
    gi, gd = vf.search(ix, torch.from_numpy(q).cuda(), qoff, qids, k, **params)
    oi, od, info = ixo.search(q, qoff, qids, k, with_info=True, **params)
    assert ix.profile_read()["scan_kernel"] == 3 and (info["method"] == 1).sum() > 256
    s = info["method"] != 2
    assert_close_with_ties(to_np(gi)[s], to_np(gd)[s], oi[s], od[s], 1e-4, "AND scan")


@pytest.mark.parametrize("dtype,dim,seg_groups", [("uint8", 128, 16), ("uint8", 192, 64), ("uint8", 80, 25), ("uint8", 992, 48),
                                                  ("float32", 100, 24), ("float32", 40, 60)])
def test_and_masks_of_the_plain_scan(dtype, dim, seg_groups):
    """The same on the 32-row kernel (uint8, and float32 of other dimensions).  Segments are as long as tuned only on lists of
    thousands of entries (short lists are cut further), which is checked: beyond 24 groups a segment takes several windows."""
    import torch
    from paper_2506_00812_amd import binding as vf
    from tests.gpu_util import assert_exact
    rng = np.random.default_rng(dim + seg_groups)
    n, T = 18_000, 17_000
    k = 64 if dim == 992 else 10
    x = rng.normal(size=(20, dim))[rng.integers(0, 20, n)] * (30 if dtype == "uint8" else 2) + rng.normal(size=(n, dim)) * (12 if dtype == "uint8" else 1)
    x = np.rint(x + 128).clip(0, 255).astype(np.uint8) if dtype == "uint8" else x.astype(np.float32)
    sizes = [17_500, 16_500, 6_500, 1537, 1536, 769, 768, 767, 33, 1]
    carry = np.zeros((n, len(sizes)), dtype=bool)
    for l, size in enumerate(sizes):
        carry[rng.permutation(n)[:size], l] = True
    off = np.concatenate([[0], np.cumsum(carry.sum(1))]).astype(np.int64)
    ids = np.nonzero(carry)[1].astype(np.int32)
    asked = [sorted(set(rng.integers(0 if j % 2 else 1, len(sizes), [1, 2, 2, 3][j % 4]).tolist())) for j in range(400)]
    qoff = np.concatenate([[0], np.cumsum([len(a) for a in asked])]).astype(np.int64)
    qids = np.array([l for a in asked for l in a], dtype=np.int32)
    q = np.ascontiguousarray(x[rng.integers(0, n, 400)])
    if dtype == "float32":
        q += 0.5 * rng.normal(size=q.shape).astype(np.float32)
    ix = vf.build_index(torch.from_numpy(x).cuda(), off, ids, len(sizes), T, 8)
    ix.tune("seg_groups", seg_groups)
    ix.tune("seg_groups_heavy", seg_groups)
    ixo = OracleIndex(x, off, ids, len(sizes), T, 8, lazy_graph=True)
    params = dict(itopk=64, width=1, iters=4, n_seeds=128)
    ix.profile_enable(True)
    vf.search(ix, torch.from_numpy(q[:16]).cuda(), np.arange(17, dtype=np.int64), np.ones(16, dtype=np.int32), k, **params)
    assert ix.profile_read()["n_scan_items"] == -(-516 // seg_groups)       # 16,500 entries in 516 groups, one tile
    for count in (400, 3):
        gi, gd = vf.search(ix, torch.from_numpy(q[:count]).cuda(), qoff[:count + 1], qids[:qoff[count]], k, **params)
        oi, od, info = ixo.search(q[:count], qoff[:count + 1], qids[:qoff[count]], k, with_info=True, **params)
        if dtype == "uint8":
            assert_exact(to_np(gi), to_np(gd), oi, od, "AND scan")
        else:
            s = info["method"] != 2
            assert_close_with_ties(to_np(gi)[s], to_np(gd)[s], oi[s], od[s], 1e-4, "AND scan")
