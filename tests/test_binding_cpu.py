"""The Python binding's own logic, without a GPU: sizes that the library computes, and the stream that calls go to."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2605_28691_amd as sk


@pytest.fixture(scope="module", autouse=True)
def built():
    import os

    if not os.path.exists(sk._LIB_PATH):
        from paper_2605_28691_amd import build

        build.build()


def test_sizes_follow_the_value_of_their_arguments():
    """Any integer-like argument counts by its present value, also after a call with the same object or an equal number."""
    want = {8: (4, 2, 32), 16: (4, 2, 64)}
    for h, shape in want.items():
        for arg in (h, np.int64(h), np.array(h), torch.tensor(h)):
            assert sk.skiparse_lse_shape(1, 2, 2, arg, 8, 64, 2, "token") == shape
            assert sk.skiparse_bwd_workspace_bytes(1, 2, 2, arg, 8, 64, 2, "token") == 4 * int(np.prod(shape))
    t = torch.tensor(8)
    assert sk.skiparse_lse_shape(1, 2, 2, t, 8, 64, 2, "token") == want[8]
    t.fill_(16)
    assert sk.skiparse_lse_shape(1, 2, 2, t, 8, 64, 2, "token") == want[16]
    assert sk.skiparse_bwd_workspace_bytes(1, 2, 2, t, 8, 64, 2, "token") == 4 * 4 * 2 * 64


def test_sizes_refuse_what_is_no_integer():
    sk.skiparse_lse_shape(1, 2, 2, 8, 8, 64, 2, "token")
    for bad in (8.0, np.float64(8), "8", None):
        with pytest.raises(ctypes.ArgumentError):
            sk.skiparse_lse_shape(1, 2, 2, bad, 8, 64, 2, "token")
        with pytest.raises(ctypes.ArgumentError):
            sk.skiparse_bwd_workspace_bytes(1, 2, 2, bad, 8, 64, 2, "token")
