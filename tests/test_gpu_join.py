"""The join kernel (self-joins of the index build) at the edges of its tiles: lists around whole groups of 32 entries and
whole tiles of 128 rows, dimensions around the contraction steps it is compiled for, candidate counts up to its 64."""
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
