"""String batches whose keys get 4, 16, 64 or 256 lanes, and batches given as a slice of a larger array of which nothing else is there (GPU only): the
base pointer lies far outside any allocation, and only bytes [offs[0], offs[n]) are backed; what a few
long strings may cost."""
import ctypes
import time

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


# one key, four, sixteen and seventeen: a step's words, one more, several steps; beside empty and short keys
@pytest.mark.parametrize("n", [1, 2, 4, 5, 16, 17, 64, 65])
@pytest.mark.parametrize("size", [0, 1, 31, 32, 127, 512, 513, 2048, 2049, 8192, 8193, 16_385, 70_003])
def test_lanes_of_a_key(mx, n, size):
    import torch

    rng = np.random.default_rng(n * size)
    for others in (size, 0, 700):
        lens = np.full(n, others, dtype=np.uint64)
        lens[rng.integers(n)] = size
        offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
        data = rng.integers(0, 256, max(int(offs[-1]), 1), dtype=np.uint8)
        got = mx.hash_str(torch.from_numpy(data).to("cuda"), torch.from_numpy(offs.view(np.int64)).to("cuda"), 7, 1000)
        assert np.array_equal(got.cpu().numpy().view(np.uint32), oracle.Oracle().hash_str(data, offs, 7, 1000))


def test_a_few_long_strings_take_little_longer_than_short_ones(mx):
    """One string of 20,000 bytes, and 16 of 1000: a microsecond or so more than one of 8, not 8 and 12."""
    import torch

    def seconds(n, size):
        data = torch.randint(0, 256, (n * size,), dtype=torch.uint8, device="cuda")
        offs = torch.arange(n + 1, dtype=torch.int64, device="cuda") * size
        edges = torch.empty((n, 3), dtype=torch.int32, device="cuda")
        lib, args = mx.lib(), (data.data_ptr(), offs.data_ptr(), n, 7, 1000, edges.data_ptr(), 0)
        best = 1.0
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(200):
                lib.mphx_hash_str(*args)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t) / 200)
        return best

    short = seconds(1, 8)
    for n, size in ((1, 20_000), (16, 1000)):
        assert seconds(n, size) < short + 3.5e-6, (n, size)
