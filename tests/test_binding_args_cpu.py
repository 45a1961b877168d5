"""Argument conversion of the Python binding (no GPU)."""
import numpy as np
import pytest
import torch

from paper_2405_17381_amd import binding


@pytest.mark.parametrize("lam", [[0.5, 0.25], (0.5, 0.25), np.array([0.5, 0.25]), np.array([0.5, 0.25], np.float32),
                                 torch.tensor([0.5, 0.25]), [torch.tensor(0.5), np.float16(0.25)], ["0.5", 0.25]])
def test_decay_rates_of_any_number_type(lam):
    assert list(binding._lam(lam, 2)) == [0.5, 0.25]
    assert list(binding._lam((x for x in lam), 2)) == [0.5, 0.25]
    for H in (1, 3):
        with pytest.raises(ValueError):
            binding._lam(lam, H)
