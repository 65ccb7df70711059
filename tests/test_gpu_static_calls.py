"""Calls on a static context make no events, streams or allocations: all of
it belongs to create.  A library loaded ahead of the HIP runtime counts the
requests that libfep3m.so makes, in a process of its own."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NAMES = {"hipEventCreateWithFlags": "void **a, unsigned b|a, b", "hipEventCreate": "void **a|a",
         "hipStreamCreateWithFlags": "void **a, unsigned b|a, b", "hipMalloc": "void **a, size_t b|a, b",
         "hipHostMalloc": "void **a, size_t b, unsigned c|a, b, c"}

RUN = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import numpy as np, torch
import paper_1503_08509_amd as fp
import workloads
x, Q = workloads.uniform(300, seed=72, charges="uniform")
x, Q = torch.from_numpy(x).cuda(), torch.from_numpy(Q).cuda()
c = fp.Context(1.0, 300, 7, static=True)
torch.cuda.synchronize()
made = shim.requests()
for _ in range(2):
    c.energy_forces(x, Q, dUdQ=True, Phi=True)
    c.energy(x, Q)
torch.cuda.synchronize()
print("requests", made, shim.requests() - made)
"""


def test_calls_on_a_static_context_request_nothing(tmp_path):
    code = '#include <cstddef>\n#include <dlfcn.h>\nstatic int count;\nextern "C" int requests() { return count; }\n' \
           'static void *real(const char *n) { return dlsym(dlopen("libamdhip64.so.7", RTLD_LAZY), n); }\n'
    for name, sig in NAMES.items():
        decl, use = sig.split("|")
        code += f'extern "C" int {name}({decl}) {{ ++count; static auto f = (int (*)({decl}))real("{name}"); return f({use}); }}\n'
    (tmp_path / "shim.cpp").write_text(code)
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", str(tmp_path / "shim.cpp"), "-o", str(tmp_path / "shim.so"), "-ldl"],
                   check=True)
    r = subprocess.run([sys.executable, "-c", RUN, str(tmp_path / "shim.so")], capture_output=True, text=True, cwd=ROOT,
                       timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    made, later = map(int, r.stdout.split("requests")[1].split())
    assert made > 0      # the library's requests are seen
    assert later == 0
