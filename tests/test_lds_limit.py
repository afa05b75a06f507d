"""The record of a kernel's LDS limit (csrc/ogc_lds_limit.h), compiled on the host: each device is raised by itself."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2301_01333_amd", "csrc")

PROGRAM = r"""
#include "ogc_lds_limit.h"
#include <stdio.h>
static OgcLdsLimit limit;
static int call(int device, size_t bytes, int rc) {   // prints 1 if the limit was raised
    int raised = 0;
    const int got = limit.raise(device, bytes, [&]() { raised = 1; return rc; });
    printf("%d%d ", raised, got);
    return got;
}
int main() {
    call(0, 100, 0);    // raised
    call(0, 100, 0);    // known
    call(0, 60, 0);     // below
    call(1, 100, 0);    // another device: raised there too
    call(0, 160, 0);    // more than before
    call(0, 160, 0);
    call(1, 160, 7);    // refused: passed on and not remembered
    call(1, 160, 0);
    call(1, 100, 0);
    call(900, 100, 0);  // no room to remember: raised every time
    call(900, 100, 0);
    call(-1, 100, 0);
    call(-1, 100, 0);
    return 0;
}
"""


def test_each_device_is_raised_by_itself(tmp_path):
    src, exe = tmp_path / "limit.cpp", tmp_path / "limit"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    assert out == ["10", "00", "00", "10", "10", "00", "17", "10", "00", "10", "10", "10", "10"]


def test_no_launch_remembers_the_limit_for_the_process():
    """Every place that raises it does so by the record above, or at every launch."""
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith((".hip", ".h", ".cpp")):
            continue
        text = open(os.path.join(CSRC, name)).read()
        for at in range(text.count("hipFuncSetAttribute(")):
            before = text.split("hipFuncSetAttribute(")[at][-400:]
            assert "limit.raise(" in before or "at every such launch" in before, name
