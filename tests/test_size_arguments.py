"""The size queries answer from their arguments' values, whatever integer type these have:
0-d arrays, and tensors that change in place between two calls."""
import numpy as np
import pytest
import torch

import paper_1512_02951_amd as sf
from paper_1512_02951_amd import pixel

QUERIES = {
    "fragments": lambda H: sf.fragment_sizes(H, 64, 1, 0x3F),
    "exceptions": lambda H: sf.exception_bytes(H, 64, 1, 0x3F, 8),
    "pixel": lambda H: pixel.fragment_sizes(H, 64, 1, 0x3F),
}


@pytest.mark.parametrize("name", QUERIES)
def test_zero_dimensional_array(name):
    assert QUERIES[name](np.array(512)) == QUERIES[name](512)
    assert QUERIES[name](np.int64(512)) == QUERIES[name](512)


@pytest.mark.parametrize("name", QUERIES)
def test_tensor_changed_in_place(name):
    H = torch.tensor(64)
    assert QUERIES[name](H) == QUERIES[name](64)
    H.fill_(512)
    assert QUERIES[name](H) == QUERIES[name](512) != QUERIES[name](64)


def test_mask_and_precision_types():
    want = sf.fragment_sizes(64, 64, 1, 0x3F, "fp16")
    assert sf.fragment_sizes(64, 64, 1, np.array(0x3F, np.uint64), "fp16") == want
    assert sf.fragment_sizes(64, 64, 1, 0x3F, np.array(sf.PRECISIONS["fp16"])) == want
