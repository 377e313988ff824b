"""String batches given as a slice of a larger array of which nothing else is there (GPU only): the
base pointer lies far outside any allocation, and only bytes [offs[0], offs[n]) are backed."""
import ctypes

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

FAR = 1 << 44  # bytes between the base pointer and the first key


@pytest.fixture(scope="module")
def mx():
    import paper_1312_0526_amd as mx

    mx.lib()
    return mx


@pytest.mark.parametrize("lens", [[8], [1], [0, 3, 0], [7], [5, 0, 2], [0, 9, 0], [16] * 63, [13] * 64 + [0],
                                  list(range(130)), [3, 2100, 0, 6, 40_001, 1]], ids=lambda x: f"{len(x)}keys{sum(x)}B")
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_only_the_slice_is_read(mx, lens, shift):
    import torch

    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
    data = np.random.default_rng(len(lens)).integers(0, 256, int(offs[-1]), dtype=np.uint8)
    n = len(lens)
    kept = torch.from_numpy(np.concatenate([np.zeros(shift, np.uint8), data])).to("cuda")  # the slice's bytes alone
    where = torch.from_numpy((offs + np.uint64(FAR + shift)).view(np.int64)).to("cuda")
    edges = torch.empty((n, 3), dtype=torch.int32, device="cuda")
    base = (kept.data_ptr() - FAR) % (1 << 64)
    rc = mx.lib().mphx_hash_str(ctypes.c_void_p(base), ctypes.c_void_p(where.data_ptr()), n, 7, 1000,
                                ctypes.c_void_p(edges.data_ptr()), ctypes.c_void_p(0))
    torch.cuda.synchronize()
    assert rc == 0
    assert np.array_equal(edges.cpu().numpy().view(np.uint32), oracle.Oracle().hash_str(data, offs, 7, 1000))
