"""What the binding does around its native part (csrc/marshal.cpp), without a GPU."""
import numpy as np
import pytest
import torch

import paper_2505_23725_amd as mlc


def test_adamw_takes_an_array_of_tensors():
    """A NumPy object array is a sequence of tuples like any other: the tensors are looked at, not the array's truth value."""
    tensors = np.empty((2, 4), dtype=object)
    for i in range(8):
        tensors[i // 4, i % 4] = torch.zeros(8)
    with pytest.raises(ValueError, match="param must live on the GPU"):
        mlc.muloco_adamw_step(tensors, mlc.AdamWHParams(lr=0.1))
