"""pxs_lower_union against a plain dictionary of positions, over every form an
input can take: dense, coordinates in any order, compressed rows and columns
with sorted or unsorted indices, entries on one side of the diagonal only or on
both with different values, different patterns of H and S, entries named twice
(their sum), real, complex, single precision and integer values.  Exact."""
import numpy as np
import pytest
import scipy.sparse as sps
import torch

from paper_1405_0194_amd import api, binding


def _expected(n, H, S):
    """H, S: dicts (r, c) -> value."""
    def low(M):
        out = {}
        for (r, c), v in M.items():
            if r < c and (c, r) not in M:
                out[(c, r)] = np.conj(v)
        out.update({k: v for k, v in M.items() if k[0] >= k[1]})
        return out
    h, s = low(H), low(S)
    keys = sorted(set(h) | set(s) | {(i, i) for i in range(n)}, key=lambda k: (k[1], k[0]))
    ptr = np.concatenate([[0], np.cumsum(np.bincount([k[1] for k in keys], minlength=n))])
    return ptr, np.array([k[0] for k in keys]), np.array([h.get(k, 0) for k in keys]), np.array([s.get(k, 0) for k in keys])


def _random(n, rng, dtype, density):
    M = {}
    for r in range(n):
        for c in range(n):
            if rng.uniform() < density:
                v = rng.integers(-9, 9) if dtype == np.int64 else rng.standard_normal()
                M[(r, c)] = dtype(v + 1j * rng.standard_normal()) if dtype == np.complex128 else dtype(v)
    return M


def _form(M, n, form, dtype, rng):
    k = list(M)
    rng.shuffle(k)
    r, c = (np.array([x[i] for x in k], dtype=np.int64) for i in (0, 1))
    v = np.array([M[tuple(x)] for x in k], dtype=dtype)
    if form == "twice":                      # every value in two parts
        coo = sps.coo_matrix((np.concatenate([v - 1, np.ones_like(v)]), (np.tile(r, 2), np.tile(c, 2))), shape=(n, n))
        csr = sps.csr_matrix((n, n), dtype=dtype)
        order = np.argsort(coo.row, kind="stable")
        csr.indptr = np.concatenate([[0], np.cumsum(np.bincount(coo.row, minlength=n))]).astype(np.int32)
        csr.indices, csr.data = coo.col[order].astype(np.int32), coo.data[order]
        return csr
    if form in ("csr_unsorted", "csc_unsorted"):
        i, j = (r, c) if form[:3] == "csr" else (c, r)
        order = np.argsort(i, kind="stable")
        ptr = np.concatenate([[0], np.cumsum(np.bincount(i, minlength=n))])
        return getattr(sps, form[:3] + "_matrix")((v[order], j[order], ptr), shape=(n, n))
    coo = sps.coo_matrix((v, (r, c)), shape=(n, n))
    if form.startswith("scipy"):
        return coo.asformat(form[6:])
    t = torch.sparse_coo_tensor(torch.from_numpy(np.stack([r, c])), torch.from_numpy(v), (n, n))
    return {"coo": lambda: t, "csr": lambda: t.coalesce().to_sparse_csr(), "csc": lambda: t.coalesce().to_sparse_csc()}[form[6:]]()


FORMS = ["scipy_coo", "scipy_csr", "scipy_csc", "csr_unsorted", "csc_unsorted", "twice", "torch_coo", "torch_csr", "torch_csc"]


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("dtype", [np.float64, np.complex128, np.float32, np.int64])
@pytest.mark.parametrize("n,density", [(1, 1.0), (7, 0.0), (9, 0.3), (23, 0.1), (16, 1.0)])
def test_every_form(form, dtype, n, density):
    if form == "twice" and dtype in (np.float32, np.float64, np.complex128) and density:
        tol = 1e-6 if dtype == np.float32 else 1e-14   # (v - 1) + 1 rounds twice
    else:
        tol = 0.0
    rng = np.random.default_rng([n, FORMS.index(form)])
    H, S = _random(n, rng, dtype, density), _random(n, rng, dtype, 0.7 * density)
    ptr, rows, hv, sv = _expected(n, H, S)
    got = api.lower_csc(_form(H, n, form, dtype, rng), _form(S, n, form, dtype, rng))
    assert got[0] == n and np.array_equal(got[1], ptr) and np.array_equal(got[2], rows)
    for x, y in ((got[3], hv), (got[4], sv)):
        assert x.dtype == (np.complex128 if dtype == np.complex128 else np.float64)
        assert np.all(np.abs(x - y) <= tol * 10)


def test_bad_lists_are_refused():
    ok = (1, np.array([0, 1, 2]), np.array([0, 1]))
    for bad in [(1, np.array([0, 1, 2]), np.array([0, 2])), (1, np.array([0, 3, 2]), np.array([0, 1])),
                (1, np.array([1, 1, 2]), np.array([0, 1])), (0, np.array([0, -1]), np.array([0, 1])),
                (2, np.array([0, 5]), np.array([0, 1, 2]))]:
        with pytest.raises(binding.PxsError):
            binding.lower_union(2, ok, bad)
    with pytest.raises(ValueError):
        binding.lower_union(3, ok, ok)
    with pytest.raises(ValueError):
        api.lower_csc(np.eye(3), np.eye(4))
