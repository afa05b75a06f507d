"""What an attention call asks of the runtime beside its launch, on the CPU: the calls are answered by a small stand-in for the
HIP runtime, which counts them (no device, nothing runs; the pointers are never read)."""
import json
import os
import subprocess
import sys

import pytest

from paper_2301_01333_amd import binding as b

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(not os.path.exists(b.LIB_PATH), reason="libogc_mlp.so not built (python -m paper_2301_01333_amd.build)")

STAND_IN = r"""
#include <stddef.h>
struct dim3 { unsigned x, y, z; };
int device, launches, raised;
size_t lds;
extern "C" {
int hipGetDevice(int* d) { *d = device; return 0; }
int hipGetLastError() { return 0; }
int hipFuncSetAttribute(const void*, int, int) { ++raised; return 0; }
int __hipPushCallConfiguration(dim3, dim3, size_t bytes, void*) { lds = bytes; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* w, size_t* bytes, void** s) { *g = *w = dim3{1, 1, 1}; *bytes = lds; *s = nullptr; return 0; }
int hipLaunchKernel(const void*, dim3, dim3, void**, size_t, void*) { ++launches; return 0; }
void set_device(int d) { device = d; }
int get_launches() { return launches; }
int get_raised() { return raised; }
size_t get_lds() { return lds; }
}
"""

CALLS = r"""
import ctypes, json, sys
runtime = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)  # before the library, whose calls then come here
runtime.get_lds.restype = ctypes.c_size_t
from paper_2301_01333_amd import binding as b
quant, out, p = b.ogc_mha_quant(0.05, 0.05, 0.05, 0.01), [], 1 << 40
for device, seq in ((0, 512), (0, 512), (0, 4096), (0, 300), (1, 512), (1, 512), (0, 512), (0, 64)):
    runtime.set_device(device)
    b.ogc_mha_run_i8(b.mha_desc(b.OGC_I8, 1, 8, seq, 128, 0.1), quant, p, p, p, p, p, 0)
    out.append([runtime.get_launches(), runtime.get_raised(), runtime.get_lds() > 65536])
print(json.dumps(out))
"""


def test_int8_attention_raises_the_lds_limit_once_per_device(tmp_path):
    src, lib = tmp_path / "runtime.cpp", tmp_path / "runtime.so"
    src.write_text(STAND_IN)
    subprocess.run(["g++", "-shared", "-fPIC", str(src), "-o", str(lib)], check=True)
    run = subprocess.run([sys.executable, "-c", CALLS, str(lib)], check=True, capture_output=True, text=True, cwd=ROOT)
    out = json.loads(run.stdout.splitlines()[-1])
    assert [o[0] for o in out] == [1, 2, 3, 4, 5, 6, 7, 8]
    assert [o[2] for o in out] == [True] * 7 + [False]
    assert [o[1] for o in out] == [1, 1, 1, 1, 2, 2, 2, 2]
