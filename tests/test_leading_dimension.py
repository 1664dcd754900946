"""The leading dimension that the Python entry points read from their operands:
a stacked tensor's last extent, the first tensor's of a list."""
import pytest
import torch

from paper_2203_09353_amd import bgemm


@pytest.mark.parametrize("x,ld", [(torch.zeros(3, 4, 5), 5), (torch.zeros(1, 1, 9), 9),
                                  (torch.zeros(4, 6, 8)[:, :, :7], 7),
                                  ([torch.zeros(4, 7), torch.zeros(2, 3)], 7)])
def test_leading_dimension(x, ld):
    assert bgemm._ld(x) == ld


@pytest.mark.parametrize("x", [torch.zeros(0, 4, 5), [], torch.zeros(3)])
def test_leading_dimension_of_nothing_is_refused(x):
    with pytest.raises(IndexError):
        bgemm._ld(x)
