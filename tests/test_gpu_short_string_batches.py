"""String batches of few keys, hashed four lanes to a key, against the oracle (GPU only): ragged blocks, arrays
shorter than a word, empty keys, keys beyond the words a quad reads, slices of a larger offset array,
and both sides of the batch size where the form changes."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mx():
    import paper_1312_0526_amd as mx

    mx.lib()
    return mx


@pytest.fixture(scope="module")
def o():
    return oracle.Oracle()


def dev(a):
    import torch

    view = {np.dtype(np.uint64): np.int64, np.dtype(np.uint8): np.uint8}[a.dtype]
    return torch.from_numpy(np.ascontiguousarray(a).view(view)).to("cuda")


def strings(lens, seed=0):
    offs = np.concatenate([[0], np.cumsum(np.asarray(lens, dtype=np.uint64))]).astype(np.uint64)
    return np.random.default_rng(seed).integers(0, 256, int(offs[-1]), dtype=np.uint8), offs


CASES = {
    "one-byte": [1], "three-bytes": [0, 3], "seven": [3, 0, 4], "eight": [8], "nine": [5, 4],
    "every-length": list(range(0, 140)),
    "block-less-one": [9] * 63, "block": [17] * 64, "block-and-one": [33] * 65,
    "near-words": [505, 511, 512, 513, 519, 520, 521, 8 * 64 * 4, 3000],
    "long-among-short": [7] * 10 + [100_003] + [61] * 60 + [2049, 70_000] + [5] * 3,
    "long-last": [12, 4097],
}


@pytest.mark.parametrize("name", list(CASES))
def test_hash_against_oracle(mx, o, name):
    data, offs = strings(CASES[name], seed=len(name))
    got = mx.hash_str(dev(data), dev(offs), 7, 1000).cpu().numpy().view(np.uint32)
    assert np.array_equal(got, o.hash_str(data, offs, 7, 1000))


@pytest.mark.parametrize("n", [1, 64, 65, 20_011, 196_608, 196_609])
def test_lookups(mx, o, n):
    import torch

    data, offs = workloads.str_keys(200_003, gen_seed=8)
    d, f = dev(data), dev(offs)
    built = mx.mphf_build_str(d, f, seed=2)
    every = mx.lookup_str(built["codes"], built["rank"], built["P"], built["seed_used"], d, f)
    assert torch.equal(torch.sort(every).values, torch.arange(200_003, device="cuda"))
    first = (200_003 - n) // 2
    part = mx.lookup_str(built["codes"], built["rank"], built["P"], built["seed_used"], d, f[first:first + n + 1])
    assert torch.equal(part, every[first:first + n])
    split = mx.hem_build(data=d, offs=f, k=9)
    whole = mx.hem_lookup(split, data=d, offs=f)
    assert torch.equal(mx.hem_lookup(split, data=d, offs=f[first:first + n + 1]), whole[first:first + n])
    values = torch.arange(200_003, device="cuda", dtype=torch.int32) % 251
    fn = mx.sf_build_str(d, f, values, 251)
    got = mx.sf_lookup_str(fn["words"], 251, fn["P"], fn["seed_used"], d, f[first:first + n + 1])
    assert torch.equal(got.to(torch.int32), values[first:first + n])
