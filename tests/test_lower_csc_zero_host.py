"""A real entry given above the diagonal only, in a pencil that is complex, is
mirrored as the conjugate of a complex number: its imaginary part is -0.0, on
the host as on the device."""
import numpy as np
import pytest
import scipy.sparse as sps
import torch

from paper_1405_0194_amd import api


@pytest.mark.parametrize("form", ["scipy", "torch", "dense"])
def test_mirrored_real_entry_of_a_complex_pencil(form):
    H = np.array([[1.0, 2.0, 0.0], [0.0, 3.0, 4.0], [0.0, 0.0, 5.0]])
    S = np.eye(3) + 1j * np.array([[0, 0.1, 0], [-0.1, 0, 0], [0, 0, 0]])
    f = {"scipy": sps.csr_matrix, "torch": lambda M: torch.from_numpy(M).to_sparse_csr(), "dense": lambda M: M}[form]
    n, colptr, rowind, hval, sval = api.lower_csc(f(H), f(S))
    cols = np.repeat(np.arange(n), np.diff(colptr))
    assert np.array_equal(hval, H.T[rowind, cols]) and np.array_equal(sval, S[rowind, cols])
    mirrored = (rowind != cols) & (hval != 0)
    assert np.count_nonzero(mirrored) == 2 and np.array_equal(np.signbit(hval.imag), mirrored)
