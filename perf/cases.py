"""Performance cases: the work a program has this library do, through its public entry points.

Every case is a dict of plain values; `listed()` names twelve, `draw(rng)` gives one more of the
same ranges.  The families:

  mphf    one MWHC minimal perfect hash of u64 or string keys (mphf_build_u64 / _str) into a
          workspace and output buffers the program keeps
  sf      one static function of u64 keys, plain or ranked layout
  hem     one HEM split of a key set into 2^k buckets
  batch   one batched build of many independent buckets with a plan the program keeps
  served  a set of build requests of mixed sizes and kinds through a build server
  peel    the layered peel of an r-uniform edge list
  lookup  the values of a batch of keys under a built function

Inputs are the library's synthetic key sets: distinct u64 keys, and printable strings with
log-normal lengths of mean 60 bytes.  Every output is whole numbers, so there is no 64-bit
reference to be nearer to: outputs are right when they are equal.
"""
import math
import random

import numpy as np
import torch

import paper_1312_0526_amd as mx

GAMMA = (123, 100)
MEAN_STR = 60.0  # mean key length in bytes


# ---- the cases -------------------------------------------------------------------------------
def listed():
    return [
        # the smallest request a build service gets: latency is all that counts
        dict(name="mphf_u64_1e3", family="mphf", keys="u64", n=1000),
        # a dictionary of strings, ragged size
        dict(name="mphf_str_20011", family="mphf", keys="str", n=20_011),
        # the ordinary build: a million integer keys
        dict(name="mphf_u64_1e6", family="mphf", keys="u64", n=1_000_000),
        # the mean size of served requests, string keys
        dict(name="mphf_str_7.8e6", family="mphf", keys="str", n=7_800_001),
        # a large integer key set
        dict(name="mphf_u64_2e27", family="mphf", keys="u64", n=1 << 27),
        # the headline's shape (strings of 60 bytes on average) at the largest size timed here
        dict(name="mphf_str_2e28", family="mphf", keys="str", n=1 << 28),
        # a static function with byte values
        dict(name="sf_u64_2e6", family="sf", n=2_000_003, sigma=256, ranked=False),
        # the HEM split with buckets of 16,384 keys on average, string keys
        dict(name="hem_str_2e26", family="hem", keys="str", n=1 << 26, k=12),
        # independent buckets of 100 to 10^6 keys, sizes log-uniform
        dict(name="batch_2048", family="batch", buckets=2048, smallest=100, largest=1_000_000, sizes=1),
        # lookups in batches of 2^16 string keys on a function of 10^7 keys
        dict(name="lookup_str_2e16", family="lookup", of="mphf", keys="str", n=10_000_000, batch=1 << 16),
        # requests of 10^3 to 10^7 keys, integers and strings, all waiting at once
        dict(name="served_24", family="served", requests=24, smallest=1000, largest=10_000_000, sizes=1),
        # the peeling order of a random 3-hypergraph just above the threshold
        dict(name="peel_1e6", family="peel", r=3, n=1_000_003, num=123),
    ]


def _log_uniform(rng, lo, hi):
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case.  Sizes are log-uniform, so they fall between the usual round numbers."""
    family = rng.choice(["mphf", "mphf", "mphf", "mphf", "sf", "hem", "batch", "lookup", "lookup", "served", "peel"])
    if family == "mphf":
        return dict(family="mphf", keys=rng.choice(["u64", "str"]), n=_log_uniform(rng, 1000, 100_000_000))
    if family == "sf":
        return dict(family="sf", n=_log_uniform(rng, 1000, 20_000_000), sigma=rng.choice([2, 3, 256, 1000, 65536, 1 << 32]),
                    ranked=rng.random() < 0.5)
    if family == "hem":
        k = rng.randint(9, 14)  # buckets of 1,000 to 60,000 keys on average
        return dict(family="hem", keys=rng.choice(["u64", "str"]), n=_log_uniform(rng, 1000 << k, min(60_000 << k, 1 << 26)), k=k)
    if family == "batch":
        return dict(family="batch", buckets=_log_uniform(rng, 16, 2048), smallest=100,
                    largest=_log_uniform(rng, 2000, 1_000_000), sizes=rng.randrange(1 << 20))
    if family == "served":
        return dict(family="served", requests=rng.randint(2, 24), smallest=1000,
                    largest=_log_uniform(rng, 10_000, 10_000_000), sizes=rng.randrange(1 << 20))
    if family == "peel":
        # vertices per edge in hundredths: just above the threshold of each r, and for r = 3 below it
        # too, where a 2-core remains
        r, num = rng.choice([(3, 123), (3, 120), (4, 133), (5, 145)])
        return dict(family="peel", r=r, n=_log_uniform(rng, 1000, 10_000_000), num=num)
    of = rng.choice(["mphf", "sf", "hem"])
    n = _log_uniform(rng, 1_000_000, 10_000_000) if of == "hem" else _log_uniform(rng, 10_000, 10_000_000)
    return dict(family="lookup", of=of, keys="u64" if of == "sf" else rng.choice(["u64", "str"]), n=n,
                batch=_log_uniform(rng, 100, n))


# ---- inputs ----------------------------------------------------------------------------------
_TABLE = None


def _length_table():
    """65,536 string lengths: quantiles of a log-normal with mean 60 and sigma 0.5 within [8, 512]."""
    global _TABLE
    if _TABLE is None:
        u = (torch.arange(65536, dtype=torch.float64) + 0.5) / 65536
        q = torch.exp(math.log(MEAN_STR) - 0.125 + 0.5 * torch.special.ndtri(u)) + 0.5
        _TABLE = torch.floor(q).clamp(8, 512).to(torch.int16).cuda()
    return _TABLE


def _keys(kind, n, seed):
    if kind == "u64":
        return (mx.gen_keys_u64(n, gen_seed=seed),)
    return mx.gen_str_keys(n, _length_table(), gen_seed=seed)


def _kind(keys):
    return mx.KEYS_U64 if keys == "u64" else mx.KEYS_STR


def _bytes(count):
    return torch.empty(max(count, 256), dtype=torch.uint8, device="cuda")


def _words(count):
    return torch.empty(max(count, 1), dtype=torch.int64, device="cuda")


def _sizes(case, count):
    """Log-uniform sizes of a batch's buckets or a server's requests: the case's, whatever the seed."""
    rng = random.Random(case["sizes"])
    return [_log_uniform(rng, case["smallest"], case["largest"]) for _ in range(count)]


def _random_edges(n, m, r, seed):
    """n edges of r distinct vertices below m: vertex q from the q-th r-th of the vertices."""
    part = m // r
    g = torch.Generator(device="cuda").manual_seed(seed)
    local = torch.randint(0, part, (n, r), dtype=torch.int32, device="cuda", generator=g)
    return (local + part * torch.arange(r, dtype=torch.int32, device="cuda")).contiguous()


def prepare(case, seed):
    family = case["family"]
    s = dict(case=case)
    if family == "mphf":
        n, m = case["n"], 3 * mx.part_size(case["n"], GAMMA)
        s["keys"] = _keys(case["keys"], n, seed)
        s["ws"] = _bytes(mx.mphf_workspace_bytes(n, GAMMA, _kind(case["keys"])))
        s["out"] = (_words((m + 31) // 32), _words((m + 511) // 512))
    elif family == "sf":
        n, sigma = case["n"], case["sigma"]
        g = torch.Generator(device="cuda").manual_seed(seed)
        s["keys"] = _keys("u64", n, seed)[0]
        s["values"] = torch.randint(0, sigma, (n,), dtype=torch.int64, device="cuda", generator=g).to(torch.int32)
        s["ws"] = _bytes(mx.sf_workspace_bytes(n, GAMMA, mx.KEYS_U64))
        if case["ranked"]:
            s["out"] = tuple(_words(w) for w in mx.sfr_sizes(n, sigma, GAMMA))
        else:
            s["out"] = _words(mx.sf_words(n, sigma, GAMMA))
    elif family == "hem":
        s["keys"] = _keys(case["keys"], case["n"], seed)
        s["ws"] = _bytes(mx.hem_workspace_bytes(case["n"], case["k"], GAMMA, _kind(case["keys"])))
        # the program's own arrays, as large as any split's tables; a split fills their start
        s["tables"] = [_words(w).zero_() for w in mx.hem_capacity(case["n"], case["k"], GAMMA)]
    elif family == "batch":
        off = np.concatenate([[0], np.cumsum(_sizes(case, case["buckets"]))]).astype(np.uint64)
        s["plan"] = mx.BatchBuild(off, gamma=GAMMA)
        s["keys"] = _keys("u64", int(off[-1]), seed)[0]
    elif family == "served":
        sizes = _sizes(case, case["requests"])
        s["server"] = mx.Server(hbm_budget=8 << 30)
        s["requests"] = [_keys("str" if i % 2 else "u64", n, seed * 64 + i) for i, n in enumerate(sizes)]
    elif family == "peel":
        s["m"] = _peel_vertices(case)
        s["edges"] = _random_edges(case["n"], s["m"], case["r"], seed)
    elif family == "lookup":
        n, batch = case["n"], case["batch"]
        keys = _keys(case["keys"], n, seed)
        if case["of"] == "sf":
            g = torch.Generator(device="cuda").manual_seed(seed)
            values = torch.randint(0, 256, (n,), dtype=torch.int32, device="cuda", generator=g)
            s["function"] = mx.sf_build_u64(keys[0], values, 256)
        elif case["of"] == "hem":
            s["function"] = mx.hem_build(*(keys if case["keys"] == "u64" else (None, *keys)), k=9)
        elif case["keys"] == "u64":
            s["function"] = mx.mphf_build_u64(*keys)
        else:
            s["function"] = mx.mphf_build_str(*keys)
        first = random.Random(seed).randrange(n - batch + 1)
        s["batch"] = (keys[0][first:first + batch],) if case["keys"] == "u64" else (keys[0], keys[1][first:first + batch + 1])
        s["out"] = _words(batch)
    return s


# ---- one pass --------------------------------------------------------------------------------
_INFO = ("P", "m", "seed_used", "tries", "n_rounds", "n_core", "frontier_total", "claims", "frontier0", "layer0")


def _with_info(d, *tensors):
    return {k: d[k] for k in _INFO + tensors}


def run(s):
    case = s["case"]
    family = case["family"]
    if family == "mphf":
        build = mx.mphf_build_u64 if case["keys"] == "u64" else mx.mphf_build_str
        return _with_info(build(*s["keys"], ws=s["ws"], out=s["out"]), "codes", "rank")
    if family == "sf":
        if case["ranked"]:
            d = mx.sfr_build_u64(s["keys"], s["values"], case["sigma"], ws=s["ws"], out=s["out"])
            fields = d["vals"]
            return dict(_with_info(d, "marks", "rank"), **({"vals": fields} if fields.numel() else {}))
        return _with_info(mx.sf_build_u64(s["keys"], s["values"], case["sigma"], ws=s["ws"], words=s["out"]), "words")
    if family == "hem":
        keys = dict(keys=s["keys"][0]) if case["keys"] == "u64" else dict(data=s["keys"][0], offs=s["keys"][1])
        d = mx.hem_build(**keys, k=case["k"], ws=s["ws"])
        for table, built in zip(s["tables"], (d["codes"], d["rank"])):
            table[:built.numel()].copy_(built)
        return dict({k: d[k] for k in ("tries", "n_rounds", "bucket_off", "code_off", "rank_off", "seeds")},
                    codes=s["tables"][0], rank=s["tables"][1])
    if family == "batch":
        plan = s["plan"]
        plan.run(s["keys"])
        return dict(codes=plan.codes, rank=plan.rank, results=plan.results)
    if family == "served":
        server = s["server"]
        tickets = [(server.submit_u64 if len(keys) == 1 else server.submit_str)(*keys) for keys in s["requests"]]
        built = [server.wait(t) for t in tickets]
        for t in tickets:
            server.release(t)
        return dict(tables=[(d["codes"], d["rank"]) for d in built],
                    found=np.array([[d["status"], d["tries"], d["n_rounds"], d["seed_used"]] for d in built], dtype=np.int64))
    if family == "peel":
        return mx.peel(s["edges"], s["m"]) if case["r"] == 3 else mx.peel_r(s["edges"], s["m"])
    f = s["function"]
    if case["of"] == "sf":
        return mx.sf_lookup_u64(f["words"], 256, f["P"], f["seed_used"], *s["batch"], out=s["out"])
    if case["of"] == "hem":
        keys = dict(keys=s["batch"][0]) if case["keys"] == "u64" else dict(data=s["batch"][0], offs=s["batch"][1])
        return mx.hem_lookup(f, **keys, out=s["out"])
    look = mx.lookup_u64 if case["keys"] == "u64" else mx.lookup_str
    return look(f["codes"], f["rank"], f["P"], f["seed_used"], *s["batch"], out=s["out"])


# ---- what a pass cannot do without -----------------------------------------------------------
def _key_bytes(keys):
    return 8.0 if keys == "u64" else MEAN_STR + 8.0


def _mphf_bytes(n):
    """Codes (2 bits a vertex) and rank samples (8 bytes per 512 vertices)."""
    m = 3 * math.ceil(n * GAMMA[0] / (3 * GAMMA[1]))
    return m / 4 + m / 64


def _peel_vertices(case):
    return case["r"] * math.ceil(case["n"] * case["num"] / (100 * case["r"]))


def work(case):
    """Keys read once, tables written once.  The arithmetic (hashing) is a few integer operations
    per key word and never bounds a pass, so no flops are claimed."""
    family = case["family"]
    if family in ("mphf", "hem"):
        nbytes = case["n"] * _key_bytes(case["keys"]) + _mphf_bytes(case["n"])
    elif family == "sf":
        bits = max(1, (case["sigma"] - 1).bit_length())
        nbytes = case["n"] * (12 + (bits + 1.25 if case["ranked"] else 1.23 * bits) / 8)
    elif family == "batch":
        nbytes = sum(8 * n + _mphf_bytes(n) for n in _sizes(case, case["buckets"]))
    elif family == "served":
        nbytes = sum(n * _key_bytes("str" if i % 2 else "u64") + _mphf_bytes(n)
                     for i, n in enumerate(_sizes(case, case["requests"])))
    elif family == "peel":
        nbytes = case["n"] * (4 * case["r"] + 10)  # edges; order, round, core mask, hinge
    else:
        # key, value, and the table bits of three vertices and a rank sample
        nbytes = case["batch"] * (_key_bytes(case["keys"]) + 8 + (3 if case["of"] == "sf" else 9))
    return {"bytes": float(nbytes), "flops": 0.0}
