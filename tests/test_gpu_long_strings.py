"""Small builds of long strings, which the build's own workgroup leaves to a hashing launch, against the oracle
(GPU only): both sides of the key length and of the total from which it does, first tries and later ones."""
import time

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

KEY, TOTAL = 512, 256 * 1024  # longest key, and bytes in all, that are hashed in the build's workgroup


@pytest.fixture(scope="module")
def mx():
    import paper_1312_0526_amd as mx

    mx.lib()
    return mx


@pytest.fixture(scope="module")
def o():
    return oracle.Oracle()


def strings(lens, seed=0):
    offs = np.concatenate([[0], np.cumsum(np.asarray(lens, dtype=np.uint64))]).astype(np.uint64)
    return np.random.default_rng(seed).integers(0, 256, int(offs[-1]), dtype=np.uint8), offs


def dev(a):
    import torch

    a = np.ascontiguousarray(a)
    return torch.from_numpy(a.view(np.int64) if a.dtype == np.uint64 else a).to("cuda")


CASES = {
    "longest": [KEY] * 30 + [9], "one-longer": [40] * 30 + [KEY + 1], "one-long": [12] * 500 + [100_000],
    "total": [256] * (TOTAL // 256), "past-total": [256] * (TOTAL // 256) + [8],
    "many": [40] * 5000, "many-past-total": [60] * 5000, "largest": [30] * 24_000,
}


@pytest.mark.parametrize("name", list(CASES))
def test_against_oracle(mx, o, name):
    data, offs = strings(CASES[name], seed=len(name))
    d, f = dev(data), dev(offs)
    tries = set()
    for seed in (0, 100, 200, 300):
        for gamma, most in (((123, 100), 64), ((119, 100), 3)):  # complete after some tries; never
            status, want = o.mphf_build_str(data, offs, seed, *gamma, max_tries=most)
            if status != oracle.OK:
                with pytest.raises(mx.MphxError) as e:
                    mx.mphf_build_str(d, f, seed=seed, gamma=gamma, max_tries=most)
                assert e.value.status == status
                assert e.value.info["tries"] == most and e.value.info["n_core"] == want["n_core"]
                continue
            got = mx.mphf_build_str(d, f, seed=seed, gamma=gamma, max_tries=most)
            tries.add(got["tries"])
            for k in ("tries", "seed_used", "n_rounds"):
                assert got[k] == want[k], k
            assert np.array_equal(got["codes"].cpu().numpy().view(np.uint64), want["words"])
            assert np.array_equal(got["rank"].cpu().numpy().view(np.uint64), want["rank"])
    assert tries


def test_long_strings_cost_their_hashing(mx):
    """2048 strings of 16,000 bytes: no more than the hashing launch of a few times over and a build of short ones."""
    import torch

    long, short = (tuple(map(dev, strings([n] * 2048))) for n in (16_000, 16))
    gamma = (2, 1)

    def seconds(f):
        best = 1.0
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            f()
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return best

    hashing = seconds(lambda: mx.hash_str(*long, 0, 1000))
    build = seconds(lambda: mx.mphf_build_str(*short, gamma=gamma))
    assert mx.mphf_build_str(*long, gamma=gamma)["tries"] == 1
    assert seconds(lambda: mx.mphf_build_str(*long, gamma=gamma)) < 2 * hashing + 2 * build + 1e-4
