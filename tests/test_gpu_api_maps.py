"""Sparse device inputs whose pattern the solver has seen take their values by
a gather on the device: equal, bit for bit, to a fresh solver's host conversion,
for every layout, real and complex, patterns given on one side only, and after
a change of pattern of the same size."""
import numpy as np
import pytest

from paper_1405_0194_amd import lattice

pytestmark = pytest.mark.gpu


def _tensors(s, layout, side, shift=0.0):
    import torch
    H, S = s.dense()
    H = H + shift * np.diag(np.arange(s.n) / s.n)
    keep = {"both": lambda M: M, "lower": np.tril, "upper": np.triu,
            "mixed": lambda M: np.where(np.add.outer(np.arange(s.n), np.arange(s.n)) % 3 == 0, np.triu(M), M)}[side]
    f = {"coo": lambda t: t.to_sparse(), "csr": lambda t: t.to_sparse_csr(), "csc": lambda t: t.to_sparse_csc()}[layout]
    return [f(torch.from_numpy(keep(M)).cuda()) for M in (H, S)]


@pytest.mark.parametrize("layout", ["coo", "csr", "csc"])
@pytest.mark.parametrize("side", ["both", "lower", "upper", "mixed"])
@pytest.mark.parametrize("hermitian", [False, True])
def test_seen_pattern_equals_a_fresh_solver(layout, side, hermitian):
    import torch
    from paper_1405_0194_amd import api
    make = lattice.make_hermitian_system if hermitian else lattice.make_system
    s = make("honeycomb", (3, 2), 5, 3.0, 42)
    kept = api.Solver()
    for step, args in enumerate([(0.0,), (0.01,), (0.02,)]):
        print("case:", layout, side, hermitian, step, flush=True)
        H, S = _tensors(s, layout, side, *args)
        a = kept.density_matrix(H, S, 0.0, lattice.BETA_300K, 20, dE=1.5)
        b = api.Solver().density_matrix(H, S, 0.0, lattice.BETA_300K, 20, dE=1.5)
        for x, y in zip(a[:-1], b[:-1]):
            assert torch.equal(x.values(), y.values()) and torch.equal(x.row_indices(), y.row_indices())
    e = next(iter(kept._cache.values()))
    assert len(e["maps"]) == 1
    # the same number of entries in other places: not taken for the seen one
    perm = np.roll(np.arange(s.n), 1)
    Hd, Sd = s.dense()
    H2, S2 = (torch.from_numpy(M[np.ix_(perm, perm)]).cuda().to_sparse_csr() for M in (Hd, Sd))
    a = kept.density_matrix(H2, S2, 0.0, lattice.BETA_300K, 20, dE=1.5)
    b = api.Solver().density_matrix(H2, S2, 0.0, lattice.BETA_300K, 20, dE=1.5)
    assert torch.equal(a[0].values(), b[0].values()) and a[-1]["N"] == b[-1]["N"]
