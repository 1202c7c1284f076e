"""CPU-only: the rows that the binding hands to the library."""
import pytest
import torch

from paper_2603_11021_amd import binding


@pytest.mark.parametrize("make", [lambda: torch.arange(6 * 48.0).reshape(6, 48)[:, :24], lambda: torch.arange(24 * 6.0).reshape(24, 6).t(),
                                  lambda: torch.arange(12 * 24.0).reshape(12, 24)[::2], lambda: torch.arange(24.0).expand(6, 24),
                                  lambda: torch.arange(6 * 24.0).reshape(2, 3, 24), lambda: torch.arange(6 * 24.0).reshape(3, 48)])
def test_rows_are_contiguous_and_the_callers(make):
    x = make()
    rows, M = binding._rows(x, 24, None)
    assert M == 6 and rows.shape == (6, 24) and rows.is_contiguous() and torch.equal(rows, x.reshape(6, 24))


def test_contiguous_rows_are_not_copied():
    x = torch.zeros(5, 24)
    assert binding._rows(x, 24, None)[0] is x
