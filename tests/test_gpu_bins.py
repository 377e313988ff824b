"""The binned record build and round 0 from degree-1 bits, against the oracle (GPU only): ragged tiles
and buckets, each bucket size, buckets that overflow (skewed edge lists, equal keys), and both sides
of the sizes where the build applies."""
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

    view = {np.dtype(np.uint64): np.int64, np.dtype(np.uint32): np.int32, np.dtype(np.uint8): np.uint8}[a.dtype]
    return torch.from_numpy(np.ascontiguousarray(a).view(view)).to("cuda")


def words(t, dtype=np.uint64):
    return t.cpu().numpy().view(dtype)


COUNTS = ("tries", "n_rounds", "frontier0", "layer0", "frontier_total")


# gamma 8 and 120 have more vertices than edges fill
@pytest.mark.parametrize("n,gamma", [(196_607, (123, 100)), (196_608, (123, 100)), (524_287, (130, 100)),
                                     (524_288, (123, 100)), (700_001, (123, 100)), (2_097_153, (123, 100)),
                                     (4_194_305, (123, 100)), (250_003, (8, 1)), (500_000, (120, 1)),
                                     (9_094_001, (123, 100))])
def test_mphf_binned(mx, o, n, gamma):
    keys = workloads.u64_keys(n, gen_seed=n)
    status, want = o.mphf_build_u64(keys, 3, *gamma)
    assert status == oracle.OK
    got = mx.mphf_build_u64(dev(keys), seed=3, gamma=gamma)
    assert np.array_equal(words(got["codes"]), want["words"])
    assert np.array_equal(words(got["rank"]), want["rank"])
    old = mx.get_option("part_build")
    mx.set_option("part_build", 0)
    try:
        other = mx.mphf_build_u64(dev(keys), seed=3, gamma=gamma)
    finally:
        mx.set_option("part_build", old)
    assert [got[k] for k in COUNTS] == [other[k] for k in COUNTS]


@pytest.mark.parametrize("n", [200_003, 2_500_001])
def test_strings_and_static_function_binned(mx, o, n):
    data, offs = workloads.str_keys(n, gen_seed=4)
    status, want = o.mphf_build_str(data, offs, 1)
    assert status == oracle.OK
    got = mx.mphf_build_str(dev(data), dev(offs), seed=1)
    assert np.array_equal(words(got["codes"]), want["words"])
    assert np.array_equal(words(got["rank"]), want["rank"])
    vals = (np.arange(n) % 251).astype(np.uint32)
    keys = workloads.u64_keys(n, gen_seed=6)
    status, want = o.sf_build_u64(keys, vals, 251, 2)
    assert status == oracle.OK
    assert np.array_equal(words(mx.sf_build_u64(dev(keys), dev(vals), 251, seed=2)["words"]), want["words"])


def _edges(kind, n, m, rng):
    if kind == "uniform":
        e = rng.integers(0, m, (n, 3))
    elif kind == "low":      # the lowest sixteenth of the vertices has all edges
        e = rng.integers(0, m // 16, (n, 3))
    elif kind == "high":     # the last, ragged bucket too
        e = m - 1 - rng.integers(0, m // 16, (n, 3))
    else:                    # path of triples: every bucket gets its edges from neighbouring tiles
        i = np.arange(n)
        e = np.stack([i % m, (i + 1) % m, (i + 2) % m], axis=1)
    bad = (e[:, 0] == e[:, 1]) | (e[:, 0] == e[:, 2]) | (e[:, 1] == e[:, 2])
    e[bad] = [0, m // 2, m - 1] if bad.sum() < 200 else np.stack([np.arange(bad.sum()) % (m - 2)] * 3, 1) + [0, 1, 2]
    return np.ascontiguousarray(e.astype(np.uint32))


@pytest.mark.parametrize("kind", ["uniform", "low", "high", "path"])
@pytest.mark.parametrize("n,m", [(200_001, 246_999), (400_003, 500_001), (1_000_000, 1_240_001), (3_000_017, 9_000_001)])
def test_peel_binned(mx, o, kind, n, m):
    e = _edges(kind, n, m, np.random.default_rng(n))
    status, want = o.peel(e, m)
    if status != oracle.OK:
        with pytest.raises(mx.MphxError) as err:
            mx.peel(dev(e), m)
        assert err.value.status == status
        return
    got = mx.peel(dev(e), m)
    assert (got["n_peeled"], got["n_rounds"]) == (want["n_peeled"], want["n_rounds"])
    for key, dt in (("order", np.uint32), ("round", np.uint32), ("core_mask", np.uint8), ("hinge", np.uint8)):
        assert np.array_equal(words(got[key], dt), want[key]), key


def test_refused_edges_and_degrees(mx):
    n, m = 250_000, 307_500
    e = _edges("uniform", n, m, np.random.default_rng(1))
    for bad in ([m, 1, 2], [5, 5, 6], [7, 0xFFFFFFFF, 8]):
        f = e.copy()
        f[n - 1] = bad
        with pytest.raises(mx.MphxError) as err:
            mx.peel(dev(f), m)
        assert err.value.status == mx.EINVAL
    for copies in (256, 200_000):  # one vertex triple: a degree above 255, a full bucket
        f = e.copy()
        f[:copies] = [3, 4, 5]
        with pytest.raises(mx.MphxError) as err:
            mx.peel(dev(f), m)
        assert err.value.status == mx.ERANGE
