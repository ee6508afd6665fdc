"""A plan's host outputs whose mapping changes between runs (the program
registers or unregisters its array): the launch writes where the array is
mapped at the time of the run.  The change is played by a stand-in for the
runtime's pointer query, which answers with another pinned array's address."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>
static const void *asked;
static void *answer;
extern "C" void tell(const void *p, void *mapped) { asked = p; answer = mapped; }
extern "C" hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
  auto real = (hipError_t(*)(hipPointerAttribute_t *, const void *))dlsym(
      dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD), "hipPointerGetAttributes");
  const hipError_t e = real(a, p);
  if (e == hipSuccess && asked && p == asked) a->devicePointer = answer;
  return e;
}
"""
CODE = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # before the runtime: its answer counts
shim.tell.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
import numpy as np, torch
import graphgen as gg, oracle
from paper_1911_09135_amd import alb
g = gg.rmat(10, 8, seed=1).with_weights(2)
gs = alb.GraphSet([g])
ref = oracle.sssp(g, 3)
a, b = (torch.full((g.n,), -7, dtype=torch.int32, pin_memory=True) for _ in range(2))
shim.tell(a.data_ptr(), b.data_ptr())
plan = alb.BatchPlan(gs, "sssp", [0], [3], outs=[a.numpy()])
for mapped_to_b in (True, False, True, False, False):
    shim.tell(a.data_ptr() if mapped_to_b else None, b.data_ptr())
    a.fill_(-7)
    b.fill_(-7)
    plan.run()
    got, other = (b, a) if mapped_to_b else (a, b)
    assert np.array_equal(got.numpy(), ref), mapped_to_b
    assert bool((other == -7).all()), mapped_to_b
plan.close()
gs.close()
print("ok")
"""


def test_outputs_are_looked_up_at_each_run(tmp_path):
    (tmp_path / "shim.cpp").write_text(SHIM)
    so = str(tmp_path / "shim.so")
    subprocess.check_call(["g++", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           str(tmp_path / "shim.cpp"), "-o", so, "-ldl"])
    env = dict(os.environ, PYTHONPATH=ROOT + os.pathsep + os.environ.get("PYTHONPATH", ""))
    r = subprocess.run([sys.executable, "-c", CODE, so], cwd=ROOT, env=env, capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
