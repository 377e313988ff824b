"""Key sets that take hundreds of peeling rounds, against the oracle: more round starts than the builds in LDS
keep there (512), and more rounds than one launch makes (1024).  The keys are picked so that their edges
form a chain: the set itself is checked on the CPU, the builds on the GPU."""
import numpy as np
import pytest

import oracle
import workloads

GAMMA = (2, 1)
SEED = 3


def chain_keys(length, tries=6):
    """`length` keys whose edges, under SEED, share a vertex of part 0 or 1 with the one before and the other
    with the one after, and have their vertex of part 2 in common with some 40 others: an edge
    leaves only once a neighbour in the chain has, from both ends."""
    o = oracle.Oracle()
    P = -(-length * GAMMA[0] // (3 * GAMMA[1]))
    hubs = np.arange(-(-length // 40))  # vertices of part 2
    for attempt in range(tries):
        keys = workloads.u64_keys(6_000_000, gen_seed=100 + attempt)
        e = o.hash_u64(keys, SEED, P).astype(np.int64)
        keep = np.isin(e[:, 2] - 2 * P, hubs)
        keys, e = keys[keep], e[keep]
        by = [np.argsort(e[:, k], kind="stable") for k in (0, 1)]
        first = [np.searchsorted(e[by[k], k], k * P + np.arange(P + 1)) for k in (0, 1)]
        used, degree, out = set(), np.zeros(len(hubs), int), []
        part, vertex = 0, 0
        used.add(0)
        while len(out) < length:
            at = by[part][first[part][vertex - part * P]:first[part][vertex - part * P + 1]]
            found = next((i for i in at if e[i, 1 - part] not in used and degree[e[i, 2] - 2 * P] < 60), None)
            if found is None:
                break
            out.append(keys[found])
            degree[e[found, 2] - 2 * P] += 1
            part, vertex = 1 - part, int(e[found, 1 - part])
            used.add(vertex)
        if len(out) == length:
            return np.array(out, dtype=np.uint64)
    raise AssertionError("no chain found")


@pytest.fixture(scope="module")
def chains():
    """Length to (keys, the oracle's build): the edges of the largest leave in more rounds than a launch makes."""
    o = oracle.Oracle()
    built = {}
    for length in (900, 1300, 2400):
        keys = chain_keys(length)
        status, want = o.mphf_build_u64(keys, SEED, *GAMMA, max_tries=1)
        assert status == oracle.OK
        built[length] = keys, want
    return built


def test_the_chains_are_long(chains):
    assert [300 < chains[n][1]["n_rounds"] for n in chains] == [True] * 3
    assert chains[900][1]["n_rounds"] < 512 < chains[1300][1]["n_rounds"] and chains[2400][1]["n_rounds"] > 1024


def dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).to("cuda")


def words(t):
    return t.cpu().numpy().view(np.uint64)


# 0: one workgroup, its round starts in LDS and then in device memory; 4, 64: groups, relaunched after 1024 rounds
@pytest.mark.gpu
@pytest.mark.parametrize("grid", [0, 4, 64])
@pytest.mark.parametrize("length", [900, 1300, 2400])
def test_single_builds(chains, length, grid):
    import paper_1312_0526_amd as mx

    keys, want = chains[length]
    old = mx.get_option("grid")
    mx.set_option("grid", grid)
    try:
        got = mx.mphf_build_u64(dev(keys), seed=SEED, gamma=GAMMA)
    finally:
        mx.set_option("grid", old)
    assert (got["tries"], got["n_rounds"]) == (1, want["n_rounds"])
    assert np.array_equal(words(got["codes"]), want["words"])
    assert np.array_equal(words(got["rank"]), want["rank"])


# a batched bucket has no room for more round starts and is left to the launch behind
@pytest.mark.gpu
def test_batched_buckets(chains):
    import torch

    import paper_1312_0526_amd as mx

    sets = [chains[n][0] for n in chains] + [workloads.u64_keys(700, gen_seed=1)] + [chains[1300][0]] * 3
    off = np.concatenate([[0], np.cumsum([len(k) for k in sets])]).astype(np.uint64)
    for shape in (dict(), dict(block=256, grid=2)):
        bb = mx.BatchBuild(off, seed=SEED, gamma=GAMMA, **shape)
        bb.run(dev(np.concatenate(sets)))
        torch.cuda.synchronize()
        res = bb.bucket_results()
        for b, keys in enumerate(sets):
            status, want = oracle.Oracle().mphf_build_u64(keys, SEED, *GAMMA)
            assert status == oracle.OK and res[b]["status"] == 0
            assert (res[b]["tries"], res[b]["n_rounds"]) == (want["tries"], want["n_rounds"]), b
            assert np.array_equal(words(bb.bucket_codes(b)), want["words"]), b
            assert np.array_equal(words(bb.bucket_rank(b)), want["rank"]), b
