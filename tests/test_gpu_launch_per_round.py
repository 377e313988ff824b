"""Rounds and layers of a launch each (option "shared_rounds"), which larger runs take by themselves, against the
oracle (GPU only): every kind of build and list, fixed and automatic grids, checks after one round and after
many, and both sides of the size where one launch takes all rounds."""
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


@pytest.fixture(params=[(0, 64), (96, 1), (0, 3)], ids=["batches-of-64", "grid-96-one-by-one", "batches-of-3"])
def launches(mx, request):
    names = ("shared_rounds", "grid", "round_batch")
    old = [mx.get_option(k) for k in names]
    for k, v in zip(names, (0, *request.param)):
        mx.set_option(k, v)
    yield
    for k, v in zip(names, old):
        mx.set_option(k, v)


def dev(a):
    import torch

    view = {np.dtype(np.uint64): np.int64, np.dtype(np.uint32): np.int32, np.dtype(np.uint8): np.uint8}[a.dtype]
    return torch.from_numpy(np.ascontiguousarray(a).view(view)).to("cuda")


def words(t, dtype=np.uint64):
    return t.cpu().numpy().view(dtype)


def same_mphf(got, want):
    assert (got["tries"], got["n_rounds"], got["n_core"]) == (want["tries"], want["n_rounds"], 0)
    assert np.array_equal(words(got["codes"]), want["words"])
    assert np.array_equal(words(got["rank"]), want["rank"])


@pytest.mark.parametrize("n", [1, 3, 1000, 20_011, 300_007, 2_200_000])
def test_mphf(mx, o, launches, n):
    keys = workloads.u64_keys(n, gen_seed=n)
    status, want = o.mphf_build_u64(keys, 5)
    assert status == oracle.OK
    same_mphf(mx.mphf_build_u64(dev(keys), seed=5), want)
    data, offs = workloads.str_keys(min(n, 300_007), gen_seed=n)
    status, want = o.mphf_build_str(data, offs, 5)
    assert status == oracle.OK
    same_mphf(mx.mphf_build_str(dev(data), dev(offs), seed=5), want)


@pytest.mark.parametrize("n,sigma", [(5, 7), (20_011, 2), (300_007, 1000), (300_007, 1 << 32)])
def test_static_function(mx, o, launches, n, sigma):
    keys = workloads.u64_keys(n, gen_seed=9)
    vals = (workloads.stream(np.uint64(3), np.arange(1, n + 1)) % np.uint64(sigma)).astype(np.uint32)
    status, want = o.sf_build_u64(keys, vals, sigma, 2)
    assert status == oracle.OK
    assert np.array_equal(words(mx.sf_build_u64(dev(keys), dev(vals), sigma, seed=2)["words"]), want["words"])
    if sigma < 1 << 32:
        vals[n // 2] = sigma
        with pytest.raises(mx.MphxError) as e:
            mx.sf_build_u64(dev(keys), dev(vals), sigma, seed=2)
        assert e.value.status == mx.EINVAL


# claim lists to the end, without one launch for their small rounds
@pytest.mark.parametrize("update_lists", [0, 16])
def test_claim_lists_alone(mx, o, launches, update_lists):
    n = 300_007
    keys = workloads.u64_keys(n, gen_seed=4)
    status, want = o.mphf_build_u64(keys, 4)
    assert status == oracle.OK
    old = mx.get_option("claim_lists"), mx.get_option("update_lists")
    mx.set_option("claim_lists", 1)
    mx.set_option("update_lists", update_lists)
    try:
        same_mphf(mx.mphf_build_u64(dev(keys), seed=4), want)
    finally:
        mx.set_option("claim_lists", old[0])
        mx.set_option("update_lists", old[1])


@pytest.mark.parametrize("r", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("n,gamma", [(1, 9.0), (20_011, 1.1), (300_007, 1.5)])
def test_peels(mx, o, launches, r, n, gamma):
    part = int(n * gamma / r) + 1
    e = np.random.default_rng(r).integers(0, part, (n, r), dtype=np.uint32) + part * np.arange(r, dtype=np.uint32)
    status, want = o.peel_r(e, r * part, r)
    assert status == oracle.OK
    for got in [mx.peel_r(dev(e), r * part)] + ([mx.peel(dev(e), r * part)] if r == 3 else []):
        assert (got["n_rounds"], got["n_peeled"]) == (want["n_rounds"], want["n_peeled"])
        for k in ("order", "round"):
            assert np.array_equal(words(got[k], np.uint32), want[k]), k
        for k in ("core_mask", "hinge"):
            assert np.array_equal(got[k].cpu().numpy(), want[k]), k


# a path takes half as many rounds as it has edges
@pytest.mark.parametrize("n", [131, 2049])
def test_path(mx, launches, n):
    e = np.stack([np.arange(n, dtype=np.uint32), np.arange(1, n + 1, dtype=np.uint32)], axis=1)
    got = mx.peel_r(dev(np.ascontiguousarray(e)), n + 1)
    i = np.arange(n)
    assert got["n_rounds"] == (n + 1) // 2 and np.array_equal(words(got["round"], np.uint32), np.minimum(i, n - 1 - i))


NAMES = ("P", "m", "seed_used", "tries", "n_rounds", "n_core", "frontier_total", "claims", "frontier0", "layer0")


@pytest.mark.parametrize("n", [4096, 4097, 262_144, 262_145])
def test_the_counters_do_not_depend_on_the_launches(mx, n):
    import torch

    keys = mx.gen_keys_u64(n, gen_seed=6)
    old = mx.get_option("shared_rounds"), mx.get_option("grid")
    mx.set_option("grid", 64)  # not in one workgroup
    try:
        got = []
        for b in (24, 18, 12, 0):
            mx.set_option("shared_rounds", b)
            got.append(mx.mphf_build_u64(keys, seed=1))
    finally:
        mx.set_option("shared_rounds", old[0])
        mx.set_option("grid", old[1])
    for g in got[1:]:
        assert [g[k] for k in NAMES] == [got[0][k] for k in NAMES]
        assert torch.equal(g["codes"], got[0]["codes"]) and torch.equal(g["rank"], got[0]["rank"])
