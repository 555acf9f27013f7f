"""The value types that the sparse-matrix call takes do not depend on what the
solver has seen: with the pattern known from an earlier call, an input is
refused or converted (bit for bit) as by a fresh solver."""
import numpy as np
import pytest

from paper_1405_0194_amd import lattice

pytestmark = pytest.mark.gpu
TAKEN = ["float64", "float32", "float16", "complex128", "complex64", "int64", "int32", "int16", "int8", "uint8", "bool",
         "conjugate"]
REFUSED = ["bfloat16", "complex32", "gradient"]


def _like(M, layout, how):
    """M (float64, CSR on the device) in a layout, with values of a type."""
    import torch
    M = {"csr": lambda: M, "csc": lambda: M.to_sparse_csc(), "coo": lambda: M.to_sparse_coo().coalesce()}[layout]()
    v = M.values() * 8.0
    if how == "conjugate":
        v = torch.complex(v, 0.0 * v).conj()
    elif how == "gradient":
        v = v.clone().requires_grad_()
    elif how in ("uint8", "bool"):
        v = v.abs().to(getattr(torch, how))
    else:
        v = v.to(getattr(torch, how))
    if layout == "csr":
        return torch.sparse_csr_tensor(M.crow_indices(), M.col_indices(), v, M.shape)
    if layout == "csc":
        return torch.sparse_csc_tensor(M.ccol_indices(), M.row_indices(), v, M.shape)
    return torch.sparse_coo_tensor(M.indices(), v, M.shape, is_coalesced=True)


@pytest.mark.parametrize("layout", ["csr", "csc", "coo"])
@pytest.mark.parametrize("how", TAKEN + REFUSED)
def test_types_are_taken_and_refused_as_by_a_fresh_solver(layout, how):
    import torch
    from paper_1405_0194_amd import api
    s = lattice.make_system("honeycomb", (3, 2), 5, 3.0, 42)
    H, S = (torch.from_numpy(M).cuda().to_sparse_csr() for M in s.dense())
    one = _like(S, layout, "float64")
    call = lambda solver, M: solver.density_matrix(M, one, 0.0, lattice.BETA_300K, 20, dE=20.0)
    print("case:", layout, how, flush=True)
    kept = api.Solver()
    call(kept, _like(H, layout, "float64"))
    assert sum(len(e["maps"]) for e in kept._cache.values()) == 1
    M = _like(H, layout, how)
    if how in REFUSED:
        with pytest.raises(Exception) as fresh:
            call(api.Solver(), M)
        with pytest.raises(Exception) as seen:
            call(kept, M)
        assert seen.type is fresh.type and str(seen.value) == str(fresh.value)
        return
    a, b = call(kept, M), call(api.Solver(), M)
    for x, y in zip(a[:-1], b[:-1]):
        assert x.dtype == y.dtype and torch.equal(x.values(), y.values())
    assert a[-1]["N"] == b[-1]["N"]
