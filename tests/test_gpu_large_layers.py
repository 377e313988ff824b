"""Peels whose large layers get launches of their own before one launch takes the rest, against the oracle
(GPU only): layers on both sides of the size where that begins, few rounds and many, each kind of list."""
import time

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

N = (1 << 22) + 1  # the smallest such run


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


NAMES = ("tries", "n_rounds", "n_core", "claims", "frontier0", "layer0")


# gamma 1.23: 10^6 edges in layer 0; 2: half of all; 30: nearly all, and hardly a round more
@pytest.mark.parametrize("n,gamma", [(N - 1, (123, 100)), (N, (123, 100)), (N, (2, 1)), (N + 2, (30, 1))])
def test_mphf(mx, o, n, gamma):
    keys = workloads.u64_keys(n, gen_seed=3)
    status, want = o.mphf_build_u64(keys, 1, *gamma)
    assert status == oracle.OK
    d = dev(keys)
    got = mx.mphf_build_u64(d, seed=1, gamma=gamma)
    assert np.array_equal(words(got["codes"]), want["words"])
    assert np.array_equal(words(got["rank"]), want["rank"])
    # the counters are those of the claim lists' rounds
    old = mx.get_option("claim_lists")
    mx.set_option("claim_lists", 20)
    try:
        lists = mx.mphf_build_u64(d, seed=1, gamma=gamma)
    finally:
        mx.set_option("claim_lists", old)
    assert [got[k] for k in NAMES] == [lists[k] for k in NAMES]


def test_mphf_that_fails(mx, o):
    keys = workloads.u64_keys(N, gen_seed=3)
    status, want = o.mphf_build_u64(keys, 1, 1, 1, max_tries=2)
    assert status == oracle.ECORE
    with pytest.raises(mx.MphxError) as e:
        mx.mphf_build_u64(dev(keys), seed=1, gamma=(1, 1), max_tries=2)
    assert e.value.status == status and e.value.info["n_core"] == want["n_core"] and e.value.info["tries"] == 2


def test_static_function(mx, o):
    n, sigma = N, 1000
    keys = workloads.u64_keys(n, gen_seed=9)
    vals = (workloads.stream(np.uint64(3), np.arange(1, n + 1)) % np.uint64(sigma)).astype(np.uint32)
    status, want = o.sf_build_u64(keys, vals, sigma, 2, 2, 1)
    assert status == oracle.OK
    got = mx.sf_build_u64(dev(keys), dev(vals), sigma, seed=2, gamma=(2, 1))
    assert np.array_equal(words(got["words"]), want["words"])


def uniform_edges(n, m, r):
    part = m // r
    return np.random.default_rng(r).integers(0, part, (n, r), dtype=np.uint32) + part * np.arange(r, dtype=np.uint32)


# 3-uniform lists without and with a 2-core; r-uniform lists
@pytest.mark.parametrize("r,hundredths", [(3, 200), (3, 100), (2, 250), (4, 133), (8, 200)])
def test_peel(mx, o, r, hundredths):
    m = r * (N * hundredths // (100 * r) + 1)
    e = uniform_edges(N, m, r)
    status, want = o.peel(e, m) if r == 3 else o.peel_r(e, m, r)
    assert status == oracle.OK
    got = mx.peel(dev(e), m) if r == 3 else mx.peel_r(dev(e), m)
    assert (got["n_rounds"], got["n_peeled"]) == (want["n_rounds"], want["n_peeled"])
    for k in ("order", "round"):
        assert np.array_equal(words(got[k], np.uint32), want[k]), k
    for k in ("core_mask", "hinge"):
        assert np.array_equal(got[k].cpu().numpy(), want[k]), k


def test_a_repeated_vertex_is_refused(mx):
    m = 3 * N
    e = uniform_edges(N, m, 3)
    e[N // 2, 1] = e[N // 2, 0]
    with pytest.raises(mx.MphxError) as err:
        mx.peel(dev(e), m)
    assert err.value.status == mx.EINVAL


def test_large_layers_take_no_longer_than_in_launches(mx):
    """2^24 keys at gamma 2, whose first layers hold most edges, against one key more, where every round has
    its own launch."""
    import torch

    def seconds(n):
        keys = mx.gen_keys_u64(n, gen_seed=5)
        ws = torch.empty(mx.mphf_workspace_bytes(n, (2, 1)), dtype=torch.uint8, device="cuda")
        best = 1.0
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            mx.mphf_build_u64(keys, seed=1, gamma=(2, 1), ws=ws)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return best

    assert seconds(1 << 24) < 1.1 * seconds((1 << 24) + 1)
