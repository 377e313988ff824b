"""Pinned host memory of the builds (GPU only), counted in a fresh process by a function in front of the
runtime's: the allocation-free build takes none, another build takes it once, and a build
that is refused it gives the same tables."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include <dlfcn.h>
#include <stddef.h>
static int (*real)(void**, size_t, unsigned);
int shim_calls, shim_refuse;
int shim_open(const char* path)
{
    void* h = dlopen(path, RTLD_NOW | RTLD_NOLOAD);
    real = h ? (int (*)(void**, size_t, unsigned))dlsym(h, "hipHostMalloc") : 0;
    return real != 0;
}
int hipHostMalloc(void** p, size_t n, unsigned flags)
{
    shim_calls++;
    return shim_refuse || !real ? 2 : real(p, n, flags);
}
"""

PROGRAM = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import torch
torch.zeros(1, device="cuda")
paths = {l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l}
assert any(shim.shim_open(p.encode()) for p in paths), paths
import paper_1312_0526_amd as mx
calls = ctypes.c_int.in_dll(shim, "shim_calls")
refuse = ctypes.c_int.in_dll(shim, "shim_refuse")

def outs(n):
    m = 3 * mx.part_size(n)
    return tuple(torch.empty(w, dtype=torch.int64, device="cuda") for w in ((m + 31) // 32, (m + 511) // 512))

def tables(d):
    return d["codes"].tolist() + d["rank"].tolist()

sizes = (1000, 300_000)
keys = [mx.gen_keys_u64(n, gen_seed=n) for n in sizes]
torch.cuda.synchronize()
calls.value = 0
want = [tables(mx.mphf_build_u64_static(k, outs(n))) for k, n in zip(keys, sizes)]
assert calls.value == 0, ("the allocation-free build took pinned memory", calls.value)
refuse.value = 1
assert [tables(mx.mphf_build_u64(k)) for k in keys] == want
assert calls.value > 0
refuse.value = calls.value = 0
assert [tables(mx.mphf_build_u64(k)) for k in keys] == want
assert calls.value == 1, calls.value
assert [tables(mx.mphf_build_u64_static(k, outs(n))) for k, n in zip(keys, sizes)] == want
assert calls.value == 1, calls.value
print("counted")
"""


def test_pinned_memory_of_the_builds(tmp_path):
    src, so = tmp_path / "shim.c", tmp_path / "libshim.so"
    src.write_text(SHIM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(so), str(src), "-ldl"], check=True)
    p = subprocess.run([sys.executable, "-c", PROGRAM, str(so)], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert p.returncode == 0 and "counted" in p.stdout, p.stderr[-2000:]
