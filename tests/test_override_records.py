"""The binding's override records (no GPU): every value numpy can make an array
of is accepted, and a batch takes one result shape per query."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2507_20667_amd import lib


def entries(rec, i, n):
    """The n complex128 entries that record i points to."""
    return np.frombuffer(ctypes.string_at(int(rec["data"][i]), 16 * n), dtype=np.complex128)


X = np.arange(6).reshape(2, 3) + 1j
VALUES = {
    "array": X,
    "complex64": X.astype(np.complex64),
    "fortran": np.asfortranarray(X),
    "list": X.tolist(),
    "tensor": torch.from_numpy(X),
    "tensor32": torch.from_numpy(X).to(torch.complex64),
    "scalars": [[complex(v) for v in row] for row in X],
    "transposed tensor": torch.from_numpy(X.T.copy()).T,
}


@pytest.mark.parametrize("a", VALUES)
@pytest.mark.parametrize("b", VALUES)
def test_override_values(a, b):
    rec, keep, first = lib._leaves([{7: VALUES[a], 2: VALUES[b]}, None])
    assert first == [0, 2, 2]
    assert rec["tensor"].tolist() == [2, 7] and (rec["dtype"] == lib.TN_C128).all()
    for i in range(2):
        assert np.array_equal(entries(rec, i, 6), X.reshape(-1))


def test_batch_needs_a_shape_per_query():
    """Too few shapes are refused before any result pointer is passed on (no
    context here: the library would refuse the call as well)."""
    with pytest.raises(IndexError):
        lib.tn_contract_batch(None, [(None, None), (None, None)], [()])
