"""Precisions and modes by every value that equals one of their names (no GPU needed)."""
import numpy as np
import pytest
import torch

from paper_2204_01722_amd import binding


@pytest.mark.parametrize("name, value", [(0, 0), ("f64", 0), ("fp64", 0), (torch.float64, 0), (1, 1), ("f32", 1),
                                         ("fp32", 1), (torch.float32, 1), (True, 1), (1.0, 1), (np.int64(1), 1),
                                         (np.str_("f32"), 1), (np.array(1), 1), (torch.tensor(1), 1),
                                         (torch.tensor(0), 0)])
def test_precision(name, value):
    assert binding._prec(name) == value


@pytest.mark.parametrize("name, value", [(0, 0), ("stored", 0), ("recompute", 1), ("initial_native", 2),
                                         ("initial_tuned", 3), ("current_20", 4), (np.int32(4), 4), (np.array(3), 3),
                                         (torch.tensor(1), 1)])
def test_mode(name, value):
    assert binding._mode(name) == value


@pytest.mark.parametrize("bad", [None, "f16", 5, -1, [], {}, (0,), torch.float16, np.array(9), torch.tensor(7)])
def test_refused(bad):
    with pytest.raises(ValueError, match="bad precision"):
        binding._prec(bad)
    with pytest.raises(ValueError, match="bad mode"):
        binding._mode(bad)
