"""Launch shapes of batched builds whose buckets are all built in LDS (GPU only): every block size and grid
gives the same tables, and none of the default grids leaves most of the device idle."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mx():
    import paper_1312_0526_amd as mx

    mx.lib()
    return mx


def plan(mx, buckets, size, **shape):
    off = np.arange(buckets + 1, dtype=np.uint64) * size
    return mx.BatchBuild(off, **shape), mx.gen_keys_u64(buckets * size, gen_seed=2)


SHAPES = [dict(block=b, grid=g) for b in (256, 512, 1024) for g in (0, 1, 64, 768)]


# the three classes of LDS; fewer buckets than compute units, more, and many times as many
@pytest.mark.parametrize("buckets,size", [(3, 900), (300, 5000), (40, 9000), (300, 18_000), (3000, 120)])
def test_every_shape_gives_the_same_tables(mx, buckets, size):
    import torch

    want = None
    for shape in SHAPES:
        bb, keys = plan(mx, buckets, size, **shape)
        bb.run(keys)
        torch.cuda.synchronize()
        got = bb.codes.clone(), bb.rank.clone(), bb.results.clone()
        if want is None:
            want = got
            assert all(r["status"] == 0 for r in bb.bucket_results())
        assert all(torch.equal(g, w) for g, w in zip(got, want)), shape


@pytest.mark.parametrize("buckets,size", [(2000, 5000), (256, 16_000)])
def test_default_grids_use_the_device(mx, buckets, size):
    import torch

    def seconds(block):
        bb, keys = plan(mx, buckets, size, block=block)
        best = 1.0
        for _ in range(8):
            torch.cuda.synchronize()
            t = time.perf_counter()
            bb.run(keys)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return best

    ref = seconds(1024)
    for block in (256, 512):
        assert seconds(block) < 1.3 * ref, block


# most of these fail a few tries, or all that they are given
@pytest.mark.parametrize("max_tries", [1, 2, 3, 20])
def test_tries_of_small_buckets(mx, max_tries):
    import torch

    sizes = [n for n in range(2, 34) for _ in range(12)]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)
    bb = mx.BatchBuild(off, max_tries=max_tries)
    keys = mx.gen_keys_u64(int(off[-1]), gen_seed=11)
    bb.run(keys)
    torch.cuda.synchronize()
    res = bb.bucket_results()
    old = mx.get_option("grid")
    mx.set_option("grid", 4)  # single builds by rounds in device memory
    try:
        seen = set()
        for b in range(len(sizes)):
            part = keys[int(off[b]):int(off[b + 1])].clone()
            try:
                want = mx.mphf_build_u64(part, seed=0, max_tries=max_tries)
                status = 0
                assert torch.equal(bb.bucket_codes(b), want["codes"]) and torch.equal(bb.bucket_rank(b), want["rank"])
            except mx.MphxError as e:
                want, status = e.info, e.status
            got = res[b]
            assert (got["status"], got["tries"], got["seed_used"], got["n_rounds"]) == \
                (status, want["tries"], want["seed_used"], want["n_rounds"]), (b, sizes[b])
            seen.add((status, int(got["tries"])))
        assert len(seen) > 1
    finally:
        mx.set_option("grid", old)
