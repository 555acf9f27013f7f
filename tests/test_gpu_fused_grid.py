"""A fused launch of one system with more workgroups than go in one grid
(2^22): 32 independent dense blocks of 363 columns, each cut into supernodes
with 330 rows below the first, at 4,096 real shifts (90 GB of factors).  The
ancestor updates of 32 supernodes are 32 x 36 tiles x 4,096 shifts, 4.7 M
workgroups, and go as two launches.  Inertia counts against the eigenvalues
(exact), at shifts midway between neighbouring eigenvalues."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_fused_updates_of_more_workgroups_than_one_grid():
    import torch
    from paper_1405_0194_amd import binding as B
    ncomp, blocks, orb, P = 32, 11, 33, 4096
    m = blocks * orb
    cols, rows = np.triu_indices(m)
    colptr = np.concatenate([[0], np.cumsum(np.tile(m - np.arange(m), ncomp))])
    rowind = np.concatenate([rows + k * m for k in range(ncomp)])
    x = np.concatenate([np.arange(blocks) + 100.0 * k for k in range(ncomp)])
    a = B.Analysis(ncomp * m, colptr, rowind, blkptr=np.arange(0, ncomp * m + 1, orb),
                   coords=np.stack([x, 0 * x, 0 * x], axis=1), leaf_cols=orb, fused_lanes=1)
    e = a.export()
    below = np.diff(e["row_ptr"]) - np.diff(e["super_ptr"])
    most = np.sort(below)[-32:]
    assert np.sum(((most + 63) // 64) ** 2) * P > 1 << 22
    rng = np.random.default_rng(8)
    H, ev = [], []
    for _ in range(ncomp):
        G = rng.standard_normal((m, m))
        M = (G + G.T) / np.sqrt(8.0 * m)
        H.append(M[rows, cols])
        ev.append(np.linalg.eigvalsh(M))
    ev = np.sort(np.concatenate(ev))
    mid = np.argsort(-np.diff(ev))[:P]       # the widest gaps
    eps = 0.5 * (ev[mid] + ev[mid + 1])
    assert np.min(np.diff(ev)[mid]) > 1e-6
    Hd = torch.from_numpy(np.concatenate(H)).cuda()
    Sd = torch.from_numpy(np.tile(np.where(rows == cols, 1.0, 0.0), ncomp)).cuda()
    print("case: 32 blocks of", m, "columns,", P, "shifts,", a.info["bytes_per_shift"] // 2 * P / 1e9, "GB", flush=True)
    torch.cuda.empty_cache()
    neg, info = B.inertia(a, Hd, Sd, eps)
    assert np.array_equal(neg, mid + 1) and np.all(info == 0)
    torch.cuda.empty_cache()
