"""Peels and assignments whose rounds share a launch, against the oracle (GPU only): group sizes
from one workgroup to the largest, lists that spill from LDS to the shared list, peels longer than
one launch's rounds, and both sides of the size where each round gets its own launch."""
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

    view = {np.dtype(np.uint64): np.int64, np.dtype(np.uint32): np.int32}[a.dtype]
    return torch.from_numpy(np.ascontiguousarray(a).view(view)).to("cuda")


def words(t, dtype=np.uint64):
    return t.cpu().numpy().view(dtype)


# grid 1: one workgroup, whose list of 4096 edges the early layers pass by far; 64 / 65: the
# barrier counts flat / in subgroups; 0 is the automatic size
@pytest.mark.parametrize("n,grid", [(1, 0), (3, 0), (511, 0), (4097, 0), (60_000, 1), (60_001, 2), (100_000, 64),
                                    (100_003, 65), (300_007, 256), (1_000_001, 0)])
def test_mphf_any_group(mx, o, n, grid):
    keys = workloads.u64_keys(n, gen_seed=n)
    status, want = o.mphf_build_u64(keys, 5)
    assert status == oracle.OK
    mx.set_option("grid", grid)
    try:
        got = mx.mphf_build_u64(dev(keys), seed=5)
    finally:
        mx.set_option("grid", 0)
    assert (got["tries"], got["n_rounds"]) == (want["tries"], want["n_rounds"])
    assert np.array_equal(words(got["codes"]), want["words"])
    assert np.array_equal(words(got["rank"]), want["rank"])


@pytest.mark.parametrize("n", [1 << 24, (1 << 24) + 1])
def test_mphf_launch_per_round_boundary(mx, o, n):
    keys = workloads.u64_keys(n, gen_seed=7)
    status, want = o.mphf_build_u64(keys, 1)
    assert status == oracle.OK
    got = mx.mphf_build_u64(dev(keys), seed=1)
    assert np.array_equal(words(got["codes"]), want["words"])
    assert np.array_equal(words(got["rank"]), want["rank"])


@pytest.mark.parametrize("sigma,grid", [(2, 1), (256, 7), (1000, 65), (1 << 32, 256)])
def test_static_function_any_group(mx, o, sigma, grid):
    n = 70_001
    keys = workloads.u64_keys(n, gen_seed=9)
    vals = (workloads.stream(np.uint64(3), np.arange(1, n + 1)) % np.uint64(sigma)).astype(np.uint32)
    status, want = o.sf_build_u64(keys, vals, sigma, 2)
    assert status == oracle.OK
    mx.set_option("grid", grid)
    try:
        got = mx.sf_build_u64(dev(keys), dev(vals), sigma, seed=2)
    finally:
        mx.set_option("grid", 0)
    assert np.array_equal(words(got["words"]), want["words"])


# a path: its two end edges leave in each round, (n + 1) / 2 rounds -- more than one launch takes
@pytest.mark.parametrize("n", [2047, 2049, 5001])
def test_path_beyond_one_launch(mx, n):
    e = np.stack([np.arange(n, dtype=np.uint32), np.arange(1, n + 1, dtype=np.uint32)], axis=1)
    got = mx.peel_r(dev(np.ascontiguousarray(e)), n + 1)
    i = np.arange(n)
    assert got["n_rounds"] == (n + 1) // 2 and got["n_peeled"] == n
    assert np.array_equal(words(got["round"], np.uint32), np.minimum(i, n - 1 - i))


# groups of several builds at once, whose members fall far behind one another
@pytest.mark.parametrize("n", [40_001, 250_003, 1_000_003])
def test_builds_side_by_side(mx, n):
    import threading

    import torch

    keys = [dev(workloads.u64_keys(n + i, gen_seed=n + i)) for i in range(6)]
    want = [mx.mphf_build_u64(k, seed=1) for k in keys]
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(8):
                got = mx.mphf_build_u64(keys[i], seed=1)
                torch.cuda.current_stream().synchronize()
                if not (torch.equal(got["codes"], want[i]["codes"]) and torch.equal(got["rank"], want[i]["rank"])):
                    wrong.append(i)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


# claim-list rounds hand small layers over to one launch and take large ones back
@pytest.mark.parametrize("n,update_lists", [(100_003, 16), (1_000_001, 16), (1_000_001, 0), (3_000_000, 1)])
def test_lists_and_one_launch_in_turn(mx, o, n, update_lists):
    keys = workloads.u64_keys(n, gen_seed=n)
    vals = (np.arange(n) % 251).astype(np.uint32)
    status, want = o.mphf_build_u64(keys, 4)
    assert status == oracle.OK
    status, sf = o.sf_build_u64(keys, vals, 251, 4)
    assert status == oracle.OK
    old = mx.get_option("claim_lists"), mx.get_option("update_lists")
    other = mx.mphf_build_u64(dev(keys), seed=4)
    mx.set_option("claim_lists", 1)
    mx.set_option("update_lists", update_lists)
    try:
        got = mx.mphf_build_u64(dev(keys), seed=4)
        fn = mx.sf_build_u64(dev(keys), dev(vals), 251, seed=4)
    finally:
        mx.set_option("claim_lists", old[0])
        mx.set_option("update_lists", old[1])
    assert [got[k] for k in ("tries", "n_rounds", "claims", "layer0")] == \
        [other[k] for k in ("tries", "n_rounds", "claims", "layer0")]
    assert np.array_equal(words(got["codes"]), want["words"])
    assert np.array_equal(words(got["rank"]), want["rank"])
    assert np.array_equal(words(fn["words"]), sf["words"])
