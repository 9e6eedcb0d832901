"""Coordinate arrays that the binding hands to the library."""
import pytest
import torch

from paper_2110_09214_amd import binding as B


@pytest.mark.parametrize("n", [1, 2, 20])
def test_contiguous_columns_are_passed_without_a_copy(n):
    """Columns of a larger structure of arrays (stride (1, capacity)) are the
    caller's own memory; other layouts have the same values in contiguous
    arrays."""
    buf = torch.rand(6, 40, dtype=torch.float64)
    x = buf[:, 3:3 + n].t()
    for k, c in enumerate(B._soa(x)):
        assert c.data_ptr() == buf[k, 3:].data_ptr() and c.is_contiguous() and c.shape == (n,)
    rows = torch.rand(2 * n, 5, dtype=torch.float64)
    for y in (rows, rows[::2], rows[:, :3], rows[:n, None, :3].transpose(1, 2), rows[:1].expand(n, 5), x[:, 1:4]):
        for k, c in enumerate(B._soa(y)):
            assert c.is_contiguous() and torch.equal(c.reshape(-1), y[:, k].reshape(-1))
    with pytest.raises(IndexError):
        B._soa(rows[:, :2])
