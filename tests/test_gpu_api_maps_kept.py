"""What a solver keeps of the patterns it has seen is bounded over all of them:
at most 16 value maps and 1 GiB of device memory (a smaller bound here), two per
pattern, the least recently used dropped first.  A dropped pattern gives the
same bits again, and the latest one is looked for first, whatever else is kept."""
import numpy as np
import pytest

from paper_1405_0194_amd import lattice

pytestmark = pytest.mark.gpu


def _pencils(count, n=24):
    """Tridiagonal pencils with one more pair of entries, each pencil at
    another place: patterns of one size that all differ."""
    import torch
    out = []
    for k in range(count):
        H = np.diag(np.linspace(-0.4, 0.4, n)) + 0.05 * (np.eye(n, k=1) + np.eye(n, k=-1))
        H[k % (n - 4) + 3 + k // (n - 4), k % (n - 4)] = H[k % (n - 4), k % (n - 4) + 3 + k // (n - 4)] = 0.01
        S = np.eye(n) + 0.02 * (np.eye(n, k=1) + np.eye(n, k=-1))
        out.append([torch.from_numpy(M).cuda().to_sparse_csr() for M in (H, S)])
    return out


def _held(solver):
    return [m for e in solver._cache.values() for m in e["maps"]]


def _bytes(maps):
    ts = [t for m in maps for t in [*m.index, *(x for q in m.maps for x in q if x is not None)]]
    return sum(t.numel() * t.element_size() for t in ts)


def _solve(solver, pencil):
    G, tr = solver.density_matrix(*pencil, 0.0, lattice.BETA_300K, 12, outputs=("rho",), dE=1.5)
    return G.values()


def test_count_and_order(monkeypatch):
    import torch
    from paper_1405_0194_amd import api
    pencils = _pencils(20)
    solver = api.Solver()
    first = []
    for k, p in enumerate(pencils):
        print("case: pattern", k, flush=True)
        first.append(_solve(solver, p))
        assert len(_held(solver)) == min(k + 1, 16)
    # the four oldest patterns were dropped; every pattern gives its bits again
    assert [len(e["maps"]) for e in solver._cache.values()] == [0] * 4 + [1] * 16
    for k in (5, 0, 19, 5):
        assert torch.equal(_solve(solver, pencils[k]), first[k])
        assert len(_held(solver)) == 16
    # the latest pattern is found by comparing its own arrays only
    calls, equal = [], torch.equal
    monkeypatch.setattr(torch, "equal", lambda a, b: calls.append(1) or equal(a, b))
    got = _solve(solver, pencils[5])
    assert len(calls) == 4 and equal(got, first[5])


def test_two_forms_of_one_pattern():
    import torch
    from paper_1405_0194_amd import api
    (H, S), = _pencils(1)
    forms = [(H, S), (H.to_sparse_csc(), S.to_sparse_csc()), (H.to_sparse_coo(), S.to_sparse_coo())]
    solver = api.Solver()
    want = _solve(api.Solver(), forms[0])
    for f in forms + forms[:1]:
        assert torch.equal(_solve(solver, f), want)
        assert len(solver._cache) == 1 and len(_held(solver)) <= 2


def test_bytes(monkeypatch):
    import torch
    from paper_1405_0194_amd import api
    pencils = _pencils(6)
    one = api.Solver()
    want = [_solve(one, p) for p in pencils]
    size = max(_bytes([m]) for m in _held(one))
    monkeypatch.setattr(api, "MAPS_BYTES", 3 * size + 1)
    solver = api.Solver()
    for p in pencils + pencils[::-1]:
        _solve(solver, p)
        assert 1 <= len(_held(solver)) <= 3 and _bytes(_held(solver)) <= 3 * size + 1
    monkeypatch.setattr(api, "MAPS_BYTES", 1)
    solver = api.Solver()
    for k, p in enumerate(pencils):
        assert torch.equal(_solve(solver, p), want[k]) and len(_held(solver)) == 1
