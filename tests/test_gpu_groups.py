"""Launches whose workgroups work through all rounds or layers as a group, where the group begins small
and grows (GPU only): every start without waiting for the grid, and a device that is busy when a
group begins.  Results against the oracle; how many joined is read from option "group_joins"."""
import threading
import time

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


@pytest.fixture(params=[0, 256], ids=["grid-auto", "grid-256"])
def at_once(mx, request):
    """Groups begin with whoever is there; yields a function that counts the joins so far."""
    old = mx.get_option("group_wait"), mx.get_option("grid")
    mx.set_option("group_wait", 0)
    mx.set_option("grid", request.param)
    mx.set_option("group_joins", 0)
    yield lambda: mx.get_option("group_joins")
    mx.set_option("group_wait", old[0])
    mx.set_option("grid", old[1])


# 30,000: layers that member 0 goes through alone; 9x10^6: lists in many spans
@pytest.mark.parametrize("n", [30_000, 100_003, 300_007, 1_000_001, 9_000_001])
def test_mphf_growing_groups(mx, o, at_once, n):
    keys = workloads.u64_keys(n, gen_seed=n)
    status, want = o.mphf_build_u64(keys, 5)
    assert status == oracle.OK
    d = dev(keys)
    for _ in range(5):
        got = mx.mphf_build_u64(d, seed=5)
        assert (got["tries"], got["n_rounds"]) == (want["tries"], want["n_rounds"])
        assert np.array_equal(words(got["codes"]), want["words"])
        assert np.array_equal(words(got["rank"]), want["rank"])
    assert at_once() > 0


@pytest.mark.parametrize("sigma", [2, 1000, 1 << 32])
def test_static_function_growing_groups(mx, o, at_once, sigma):
    n = 300_001
    keys = workloads.u64_keys(n, gen_seed=9)
    vals = (workloads.stream(np.uint64(3), np.arange(1, n + 1)) % np.uint64(sigma)).astype(np.uint32)
    status, want = o.sf_build_u64(keys, vals, sigma, 2)
    assert status == oracle.OK
    for _ in range(5):
        got = mx.sf_build_u64(dev(keys), dev(vals), sigma, seed=2)
        assert np.array_equal(words(got["words"]), want["words"])
    assert at_once() > 0


# claim-list rounds and shared rounds in turn, the layers above in a launch of their own
def test_lists_growing_groups(mx, o, at_once):
    n = 1_000_003
    keys = workloads.u64_keys(n, gen_seed=n)
    status, want = o.mphf_build_u64(keys, 4)
    assert status == oracle.OK
    old = mx.get_option("claim_lists")
    mx.set_option("claim_lists", 1)
    try:
        for _ in range(5):
            got = mx.mphf_build_u64(dev(keys), seed=4)
            assert np.array_equal(words(got["codes"]), want["words"])
            assert np.array_equal(words(got["rank"]), want["rank"])
    finally:
        mx.set_option("claim_lists", old)
    assert at_once() > 0


# skewed: the buckets overflow and a group adds the edges up
@pytest.mark.parametrize("skew,n", [(1.0, 250_001), (1.2, 300_001), (1.2, 3_000_001)])
def test_peel_growing_groups(mx, o, at_once, skew, n):
    rng = np.random.default_rng(n)
    part = (2 * n + 2) // 3
    e = (rng.random((n, 3)) ** skew * part).astype(np.uint32) + part * np.arange(3, dtype=np.uint32)
    want = o.peel(e, 3 * part)
    assert want[0] == oracle.OK
    d = dev(e)
    for _ in range(5):
        got = mx.peel(d, 3 * part)
        for k in ("order", "round"):
            assert np.array_equal(words(got[k], np.uint32), want[1][k]), k
        assert np.array_equal(got["core_mask"].cpu().numpy(), want[1]["core_mask"])
    assert at_once() > 0


# rounds beyond one launch, one edge each way: the group grows when hardly any work is left for it
@pytest.mark.parametrize("n", [2049, 5001])
def test_path_growing_groups(mx, at_once, n):
    e = np.stack([np.arange(n, dtype=np.uint32), np.arange(1, n + 1, dtype=np.uint32)], axis=1)
    got = mx.peel_r(dev(np.ascontiguousarray(e)), n + 1)
    i = np.arange(n)
    assert got["n_rounds"] == (n + 1) // 2 and got["n_peeled"] == n
    assert np.array_equal(words(got["round"], np.uint32), np.minimum(i, n - 1 - i))


def test_a_busy_device_does_not_keep_a_group_small(mx):
    """A build that finds all but two compute units taken for a millisecond is delayed by about that, whenever
    the others are taken."""
    import torch

    n = 9_000_000
    keys = mx.gen_keys_u64(n, gen_seed=5)
    want = mx.mphf_build_u64(keys, seed=1)
    ws = torch.empty(mx.mphf_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    out = tuple(torch.empty_like(want[k]) for k in ("codes", "rank"))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    # as many workgroups as compute units less two, each with nearly all of one's LDS
    off = np.arange(8 * (cus - 2) + 1, dtype=np.uint64) * 18_000
    plan = mx.BatchBuild(off, grid=cus - 2)
    bucket_keys = mx.gen_keys_u64(int(off[-1]), gen_seed=2)
    streams = torch.cuda.Stream(), torch.cuda.Stream()

    def batch():
        with torch.cuda.stream(streams[0]):
            plan.run(bucket_keys)

    def build():
        with torch.cuda.stream(streams[1]):
            return mx.mphf_build_u64(keys, seed=1, ws=ws, out=out)

    def seconds(f):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        return time.perf_counter() - t

    alone, busy = (min(seconds(f) for _ in range(4)) for f in (build, batch))
    took = []
    for delay in np.arange(0.0, 1.8e-3, 1e-4):
        go = threading.Event()

        def later():
            go.wait()
            t = time.perf_counter()
            while time.perf_counter() - t < delay:
                pass
            batch()

        other = threading.Thread(target=later)
        other.start()
        go.set()
        t = time.perf_counter()
        got = build()
        took.append(time.perf_counter() - t)
        other.join()
        torch.cuda.synchronize()
        assert torch.equal(got["codes"], want["codes"]) and torch.equal(got["rank"], want["rank"])
    assert np.median(took) < 2 * (alone + busy) + 2e-3, (alone, busy, took)
