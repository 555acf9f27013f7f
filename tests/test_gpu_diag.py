"""The diagonal-block kernels over their widths: blocks of 16 columns with
every kind of remainder, alone (a dense pencil is one panel) and as the panels
of a wider supernode.  Selected inverses and pivots against the dense inverse
and determinant, inertia counts against the eigenvalues (exact); bar of the
other GPU tests, |x - y| <= 1e-10 max(|y|, 1e-3 max|y|).
"""
import numpy as np
import pytest

from oracle import dense as odense

pytestmark = pytest.mark.gpu
TOL = 1e-10


@pytest.mark.parametrize("n,panel", [(1, 64), (2, 64), (15, 64), (16, 64), (17, 64), (31, 64), (33, 64), (48, 64),
                                     (49, 64), (63, 64), (64, 64), (65, 64), (130, 64), (97, 31), (50, 17), (40, 1)])
@pytest.mark.parametrize("hermitian", [False, True])
def test_dense_pencil(n, panel, hermitian):
    import scipy.linalg as sla
    import torch
    from paper_1405_0194_amd import binding as B
    rng = np.random.default_rng(n * 100 + panel)
    G = rng.standard_normal((2, n, n)) + (1j * rng.standard_normal((2, n, n)) if hermitian else 0.0)
    H, S = G[0] + G[0].conj().T, 0.1 * (G[1] + G[1].conj().T)
    H /= np.abs(H).sum(axis=1).max()
    S += np.diag(1.0 + np.abs(S).sum(axis=1))
    cols, rows = np.triu_indices(n)          # column-major lower triangle
    colptr = np.concatenate([[0], np.cumsum(n - np.arange(n))])
    print("case: dense", n, "panel", panel, "hermitian", hermitian, flush=True)
    a = B.Analysis(n, colptr, rows, leaf_cols=n, panel_width=panel)
    Hd, Sd = (torch.from_numpy(np.ascontiguousarray(M[rows, cols])).cuda() for M in (H, S))
    w = rng.uniform(-0.5, 0.5, 5) + 1j * rng.uniform(0.02, 0.4, 5)
    f = (B.HermitianFactorization if hermitian else B.Factorization)(a, Hd, Sd, w)
    assert np.all(f.info == 0)
    d = [f.diag(l).cpu().numpy() for l in range(5)]
    f.selinv()
    for l in range(5):
        A = H - w[l] * S
        Z = np.linalg.inv(A)
        assert float(np.max(odense.entry_error(f.selected(l).cpu().numpy(), Z[rows, cols]))) <= TOL
        # product of the pivots: the determinant (n multiplications)
        sign, logdet = np.linalg.slogdet(A)
        assert abs(np.sum(np.log(np.abs(d[l]))) - logdet) <= 1e-10 * max(1.0, n)
        assert abs(np.prod(d[l] / np.abs(d[l])) - sign) <= 1e-10
    ev = sla.eigvalsh(H, S)
    eps = np.concatenate([[ev[0] - 0.1, ev[-1] + 0.1], 0.5 * (ev[1:] + ev[:-1])[:6]])
    neg, info = (B.inertia_hermitian if hermitian else B.inertia)(a, Hd, Sd, eps)
    assert np.array_equal(neg, [int(np.sum(ev < e)) for e in eps]) and np.all(info == 0)


@pytest.mark.parametrize("dims,orb,akw", [
    (40, 4, dict(leaf_cols=64)), (33, 3, dict(leaf_cols=20, panel_width=7)), (50, 13, dict(leaf_cols=100)),
    (30, 13, dict(leaf_cols=128, panel_width=48)), (20, 1, dict(leaf_cols=4)), (25, 17, dict(leaf_cols=64))])
@pytest.mark.parametrize("fused", [1, -1])
def test_chains_of_small_supernodes(dims, orb, akw, fused):
    """Panels with at most 64 rows below (their rows and their selected
    inverse in one workgroup), and supernodes just over that."""
    import torch
    from paper_1405_0194_amd import binding as B
    from paper_1405_0194_amd import lattice
    s = lattice.make_system("chain", dims, orb, 2.0, 9)
    Hd, Sd = s.dense()
    rng = np.random.default_rng(dims)
    w = rng.uniform(-0.6, 0.6, 11) + 1j * rng.uniform(0.02, 0.5, 11)
    print("case: chain", dims, orb, akw, "fused", fused, flush=True)
    a = B.Analysis.from_system(s, fused_lanes=fused, **akw)
    H, S = torch.from_numpy(s.hval).cuda(), torch.from_numpy(s.sval).cuda()
    f = B.Factorization(a, H, S, w)
    assert np.all(f.info == 0)
    f.selinv()
    cols = s.entry_cols()
    for l in (0, 5, 10):
        Z = odense.shifted_inverse(Hd, Sd, w[l])
        assert float(np.max(odense.entry_error(f.selected(l).cpu().numpy(), Z[s.rowind, cols]))) <= TOL
    ev = np.sort(odense.gen_eigh(Hd, Sd)[0])
    eps = 0.5 * (ev[1:] + ev[:-1])[:: max(1, len(ev) // 7)]
    neg, info = B.inertia(a, H, S, eps)
    assert np.array_equal(neg, [int(np.sum(ev < e)) for e in eps]) and np.all(info == 0)
