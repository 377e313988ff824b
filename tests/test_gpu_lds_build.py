"""Builds whose hypergraph lives in LDS -- single small builds and the buckets of batched launches --
and the code table that larger buckets keep partly in LDS, against the oracle (GPU only), at the
edges of what fits."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

STATE = 2352  # bytes of LDS beside the vertices'


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

    a = np.ascontiguousarray(a)
    return torch.from_numpy(a.view(np.int64) if a.dtype == np.uint64 else a).to("cuda")


def words(t):
    return t.cpu().numpy().view(np.uint64)


def keys_with(m):
    """The most keys with at most m vertices at gamma = 1.23."""
    n = m * 100 // 123
    while 3 * (((n + 1) * 123 + 299) // 300) <= m:
        n += 1
    return n


# 24 KB with 256 threads; 158 KB with the queue in LDS (7 bytes a vertex) and without (5 bytes)
EDGES = sorted({keys_with((b * 1024 - STATE) // per) + d for b, per in ((24, 7), (158, 7), (158, 5)) for d in (-8, 0, 8)}
               | {2, 64, 2048, 2049})


@pytest.mark.parametrize("n", EDGES)
@pytest.mark.parametrize("kind", ["u64", "str"])
def test_small_build_edges(mx, o, n, kind):
    if kind == "u64":
        keys = (workloads.u64_keys(n, gen_seed=n),)
        status, want = o.mphf_build_u64(*keys, seed=3)
        build = mx.mphf_build_u64
    else:
        keys = workloads.str_keys(n, gen_seed=n)
        status, want = o.mphf_build_str(*keys, seed=3)
        build = mx.mphf_build_str
    if status != oracle.OK:  # two keys never peel
        with pytest.raises(mx.MphxError) as e:
            build(*map(dev, keys), seed=3)
        assert e.value.status == status and e.value.info["tries"] == 64 and e.value.info["n_core"] == want["n_core"]
        return
    got = build(*map(dev, keys), seed=3)
    for k in ("tries", "seed_used", "n_rounds", "P"):
        assert got[k] == want[k], k
    assert got["n_core"] == 0 and got["claims"] >= n and got["frontier_total"] >= got["claims"]
    assert np.array_equal(words(got["codes"]), want["words"])
    assert np.array_equal(words(got["rank"]), want["rank"])


def test_small_build_counts_equal_the_general_path(mx):
    """The info's counters do not depend on the path ("grid" selects the general one)."""
    names = ("P", "m", "seed_used", "tries", "n_rounds", "n_core", "frontier_total", "claims", "frontier0", "layer0")
    for n in (5, 777, 9000, 25_000):
        keys = dev(workloads.u64_keys(n, gen_seed=n))
        small = mx.mphf_build_u64(keys, seed=1)
        mx.set_option("grid", 4)
        try:
            general = mx.mphf_build_u64(keys, seed=1)
        finally:
            mx.set_option("grid", 0)
        assert [small[k] for k in names] == [general[k] for k in names], n


# copies of one key: degrees a state byte cannot hold (64 and more), then ones no record can (256)
@pytest.mark.parametrize("copies", [2, 63, 64, 100, 255, 256])
def test_small_build_dense_vertices(mx, o, copies):
    keys = np.concatenate([workloads.u64_keys(3000, gen_seed=4), np.full(copies, 12345, np.uint64)])
    status, want = o.mphf_build_u64(keys, seed=0, max_tries=3)
    assert status in (oracle.EDUP, oracle.ERANGE)
    with pytest.raises(mx.MphxError) as e:
        mx.mphf_build_u64(dev(keys), seed=0, max_tries=3)
    assert e.value.status == status
    assert e.value.info["tries"] == (3 if status == oracle.EDUP else 1)


def batch(mx, sets, **shape):
    import torch

    off = np.concatenate([[0], np.cumsum([len(k) for k in sets])]).astype(np.uint64)
    bb = mx.BatchBuild(off, max_tries=8, **shape)
    bb.run(dev(np.concatenate(sets)))
    torch.cuda.synchronize()
    return bb, bb.bucket_results()


# alone: every bucket fits, a launch of LDS builds alone; else larger buckets go first
@pytest.mark.parametrize("alone", [True, False])
@pytest.mark.parametrize("block,kb", [(256, 48), (512, 78), (1024, 158)])
def test_batched_lds_edges(mx, o, block, kb, alone):
    edge = keys_with((kb * 1024 - STATE) // 7)
    sizes = [1, 100, edge - 8, edge, 5000] + ([] if alone else [edge + 8, 60_000])
    sets = [workloads.u64_keys(n, gen_seed=n + 1) for n in sizes]
    sets.append(np.concatenate([workloads.u64_keys(900, gen_seed=2), np.full(80, 7, np.uint64)]))   # left: a 2-core
    sets.append(np.concatenate([workloads.u64_keys(900, gen_seed=3), np.full(300, 7, np.uint64)]))  # left: degree 300
    bb, res = batch(mx, sets, block=block)
    for b, keys in enumerate(sets):
        status, want = o.mphf_build_u64(keys, seed=0, max_tries=8)
        assert res[b]["status"] == (oracle.ECORE if status == oracle.EDUP else status), b
        assert res[b]["tries"] == want["tries"], b
        if status == oracle.OK:
            assert res[b]["n_rounds"] == want["n_rounds"], b
            assert np.array_equal(words(bb.bucket_codes(b)), want["words"]), b
            assert np.array_equal(words(bb.bucket_rank(b)), want["rank"]), b


@pytest.mark.parametrize("block,vertices", [(256, 196_608), (512, 319_488), (1024, 647_168)])
def test_batched_codes_partly_in_lds(mx, o, block, vertices):
    edge = keys_with(vertices)
    sizes = [edge - 200, edge, edge + 3, edge + 5000]
    sets = [workloads.u64_keys(n, gen_seed=n + 1) for n in sizes]
    bb, res = batch(mx, sets, block=block)
    for b, keys in enumerate(sets):
        status, want = o.mphf_build_u64(keys, seed=0)
        assert status == oracle.OK and res[b]["status"] == 0
        assert np.array_equal(words(bb.bucket_codes(b)), want["words"]), b
        assert np.array_equal(words(bb.bucket_rank(b)), want["rank"]), b


# the last strings of an array, where a read of whole words would pass its end
@pytest.mark.parametrize("first", [0, 1, 2, 3])
def test_strings_at_the_end_of_the_array(mx, o, first):
    rng = np.random.default_rng(first)
    for last in list(range(0, 40)) + [63, 64, 65, 100]:
        lens = np.array([first + 5, 9, 31, 32, 33, 70, 36, last + 6], dtype=np.uint64)
        offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
        data = rng.integers(0, 256, int(offs[-1]), dtype=np.uint8)
        status, want = o.mphf_build_str(data, offs, 1)
        assert status == oracle.OK
        got = mx.mphf_build_str(dev(data), dev(offs), seed=1)
        assert got["tries"] == want["tries"]
        assert np.array_equal(words(got["codes"]), want["words"])
