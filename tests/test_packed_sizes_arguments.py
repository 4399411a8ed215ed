"""The Python calls for packed sizes take and refuse the same arguments whatever was asked before."""
import ctypes

import numpy as np
import pytest

import paper_2306_00978_amd as awq


@pytest.mark.parametrize("name,group", [("awq_packed_sizes", 128), ("awq_packed_sizes_w3", 128), ("awq_packed_sizes_w2", 64)])
def test_only_ints_are_taken(name, group):
    fn = getattr(awq, name)
    sizes = fn(4096, 1024)
    assert sizes == fn(4096, 1024, group) == fn(N=4096, K=1024, group=group) == fn(np.int64(4096), 1024)
    assert fn(np.array(4096), 1024) == sizes                # no hash, but an index
    for bad in ((4096.0, 1024), (4096, 1024.0), (4096, 1024, float(group)), ("4096", 1024), ([4096], 1024)):
        with pytest.raises(ctypes.ArgumentError):
            fn(*bad)
    for _ in range(2):
        with pytest.raises(awq.AwqError):
            fn(4096, 1000)
