"""The tile products at the widths the library picks by launch size.

A launch with few shifts runs 16- or 32-row tiles, one with many 64-row
tiles; panels whose rows below end inside a tile, whose columns end inside a
stage (8 complex, 16 real), and whose Z_BB crosses from the supernode's own columns to the
rows below it at a position that is no multiple of 8 take every path of the
operand loads.  Selected inverses against the dense inverse of the oracle, at
the parity bar of the other GPU tests (|x - y| <= 1e-10 max(|y|, 1e-3 max|y|));
the real products by the inertia counts against the eigenvalues (exact).
"""
import numpy as np
import pytest

from oracle import dense as odense
from paper_1405_0194_amd import lattice

pytestmark = pytest.mark.gpu
TOL = 1e-10


@pytest.mark.parametrize("nshift", [1, 9, 70, 300])
@pytest.mark.parametrize("kind,dims,orb,cut,akw", [
    ("honeycomb", (4, 4), 13, 3.0, {}),
    ("cubic", (4, 4, 3), 13, 2.0, dict(panel_width=23, leaf_cols=40)),
    ("cubic", (4, 3, 3), 9, 2.0, dict(panel_width=61, selinv_streams=1)),
    ("chain", 97, 3, 2.0, dict(panel_width=7, leaf_cols=33)),
])
@pytest.mark.parametrize("hermitian", [False, True])
def test_selected_inverse_by_number_of_shifts(kind, dims, orb, cut, akw, nshift, hermitian):
    import torch
    from paper_1405_0194_amd import binding as B
    make = lattice.make_hermitian_system if hermitian else lattice.make_system
    s = make(kind, dims, orb, cut, 77)
    Hd, Sd = s.dense()
    rng = np.random.default_rng(nshift)
    w = rng.uniform(-0.6, 0.6, nshift) + 1j * rng.uniform(0.02, 0.5, nshift)
    print("case:", kind, dims, s.n, akw, "shifts", nshift, "hermitian", hermitian, flush=True)
    a = B.Analysis.from_system(s, **akw)
    H, S = torch.from_numpy(s.hval).cuda(), torch.from_numpy(s.sval).cuda()
    f = (B.HermitianFactorization if hermitian else B.Factorization)(a, H, S, w)
    assert np.all(f.info == 0)
    f.selinv()
    cols = s.entry_cols()
    for l in sorted({0, nshift // 2, nshift - 1}):
        Z = odense.shifted_inverse(Hd, Sd, w[l])
        assert float(np.max(odense.entry_error(f.selected(l).cpu().numpy(), Z[s.rowind, cols]))) <= TOL
        if hermitian:
            zu = f.selected(l, upper=True).cpu().numpy()
            assert float(np.max(odense.entry_error(zu, Z[cols, s.rowind]))) <= TOL


@pytest.mark.parametrize("nshift", [1, 9, 70, 300])
@pytest.mark.parametrize("kind,dims,orb,cut,akw", [
    ("honeycomb", (4, 4), 13, 3.0, {}),
    ("cubic", (4, 4, 3), 13, 2.0, dict(panel_width=23, leaf_cols=40)),
    ("cubic", (4, 3, 3), 9, 2.0, dict(panel_width=61)),
    ("chain", 97, 3, 2.0, dict(panel_width=7, leaf_cols=33, fused_lanes=1)),
])
def test_inertia_by_number_of_shifts(kind, dims, orb, cut, akw, nshift):
    import scipy.linalg as sla
    import torch
    from paper_1405_0194_amd import binding as B
    s = lattice.make_system(kind, dims, orb, cut, 78)
    Hd, Sd = s.dense()
    ev = sla.eigh(Hd, Sd, eigvals_only=True)
    gaps = np.diff(ev)
    # middles of the widest gaps, well away from every eigenvalue
    eps = (0.5 * (ev[1:] + ev[:-1]))[np.argsort(-gaps)[:max(1, len(gaps) // 2)]]
    eps = np.resize(eps, nshift)
    print("case: inertia", kind, dims, s.n, akw, "shifts", nshift, flush=True)
    a = B.Analysis.from_system(s, **akw)
    neg, info = B.inertia(a, torch.from_numpy(s.hval).cuda(), torch.from_numpy(s.sval).cuda(), eps)
    assert np.array_equal(neg, [int(np.sum(ev < e)) for e in eps]) and np.all(info == 0)
