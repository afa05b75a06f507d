"""Builds libogc_mlp.so (gfx950 kernels + C ABI) in-tree with hipcc.  `python -m paper_2301_01333_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libogc_mlp.so")
SOURCES = ["ogc_kernels.hip", "ogc_mha.hip", "ogc_mha_i8.hip", "ogc_api.cpp"]


FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         # packed fp32 VALU ops are kept off for every HIP translation unit in this repository
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed (%d)\n%s" % (r.returncode, out))
    return out


def build_library(verbose: bool = True) -> str:
    """Compiles every source to an object (in parallel, one hipcc each) and links the shared library."""
    import tempfile
    from concurrent.futures import ThreadPoolExecutor

    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + ".tmp.%d" % os.getpid()
    with tempfile.TemporaryDirectory() as td:
        objs = [os.path.join(td, os.path.splitext(s)[0] + ".o") for s in SOURCES]
        cmds = [[hipcc] + FLAGS + ["-c", os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objs)]
        with ThreadPoolExecutor(len(cmds)) as pool:
            outs = list(pool.map(lambda c: _run(c, verbose), cmds))
        try:
            outs.append(_run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", tmp], verbose))
        except RuntimeError:
            if os.path.exists(tmp):
                os.remove(tmp)
            raise
    if verbose and os.environ.get("OGC_BUILD_WARNINGS"):
        print("\n".join(o for o in outs if o.strip()), flush=True)
    os.replace(tmp, LIB)
    return LIB


def _device_assembly(source: str) -> str:
    import tempfile

    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as td:
        out = os.path.join(td, "k.s")
        cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off", "-Xclang", "-target-feature",
               "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-S", "--cuda-device-only",
               "-o", out, os.path.join(CSRC, source)]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if r.returncode != 0:
            raise RuntimeError("hipcc -S failed\n" + r.stdout)
        with open(out) as f:
            return f.read()


def check_stream_kernel_registers(verbose: bool = True) -> None:
    """The stream kernel keeps its operands and accumulators in v80..v255 behind the compiler's back
    (amdgpu_num_vgpr caps the compiler below v80).  This compiles the kernels to assembly and fails if any
    compiler-generated instruction of those kernels WRITES a register at or above v80, reads one outside the
    accumulator range v128..v255 (the epilogue takes the accumulators as sources where they are), or if the
    kernels contain calls."""
    import re

    text = _device_assembly("ogc_kernels.hip")
    reg = re.compile(r"\bv(\d+)\b|\bv\[(\d+):(\d+)\]")
    checked = 0
    for m in re.finditer(r"^(_Z20ogc_layer_dma_kernel\w*):[^\n]*\n(.*?)\n\ts_endpgm", text, re.S | re.M):
        name, body = m.group(1), m.group(2)
        in_asm = False
        for line in body.splitlines():
            if "#ASMSTART" in line:
                in_asm = True
            elif "#ASMEND" in line:
                in_asm = False
            elif not in_asm:
                code = line.split(";")[0]
                if "s_swappc" in code or "s_setpc" in code:
                    raise RuntimeError("%s contains a call: %s" % (name, line.strip()))
                parts = code.strip().split(None, 1)
                if len(parts) < 2:
                    continue
                mnem, ops = parts[0], [o.strip() for o in parts[1].split(",")]
                stores = mnem.startswith(("global_store", "scratch_store", "buffer_store", "flat_store", "ds_write", "ds_add",
                                          "global_atomic", "s_"))
                for i, op in enumerate(ops):
                    for a, b, c in reg.findall(op):
                        lo, hi = (int(a), int(a)) if a else (int(b), int(c))
                        if hi < 80:
                            continue
                        is_dst = i == 0 and not stores
                        if is_dst or lo < 128:
                            raise RuntimeError("%s: compiler code %s v%d..v%d, which the hand-scheduled loop owns: %s" % (
                                name, "writes" if is_dst else "reads", lo, hi, line.strip()))
        checked += 1
    if checked == 0:
        raise RuntimeError("no stream kernels found in the assembly")
    # Kernels with one fixed epilogue (last template argument 1, 3, 4: ReLU / no activation / GELU with a requantized
    # result, and 2: split-K partials) must not touch scratch memory: a reload of a spilled register in the code between
    # the assembly blocks makes the compiler wait for every outstanding vector-memory operation, the ring's direct loads
    # included (a third more time per launch when it happened).
    spilling = 0
    for m in re.finditer(r"\.name:\s+(_Z20ogc_layer_dma_kernel\w+)\s*\n\s+\.private_segment_fixed_size:\s+(\d+)", text):
        name, scratch = m.group(1), int(m.group(2))
        fixed = re.search(r"Li([1-4])EEv", name)
        if scratch > 0:
            spilling += 1
            if fixed:
                raise RuntimeError("%s uses %d bytes of scratch memory per lane (register spills)" % (name, scratch))
    # The fused chain's pair kernel is for two workgroups on a CU: 128 registers, none of them spilled.
    pairs = re.findall(r"\.name:\s+(_Z\d+ogc_fused_chain_pair_kernel\w+)\s*\n\s+\.private_segment_fixed_size:\s+(\d+)", text)
    if len(pairs) != 4 or any(int(scratch) for _, scratch in pairs):
        raise RuntimeError("fused pair kernels (name, bytes of scratch memory per lane): %s" % pairs)
    # Its streaming kernel counts on weights that arrive in order: a reload of a spilled register would wait for all of them.
    streams = re.findall(r"\.name:\s+(_Z\d+ogc_fused_chain_stream_kernel\w+)\s*\n\s+\.private_segment_fixed_size:\s+(\d+)", text)
    if len(streams) != 3 or any(int(scratch) for _, scratch in streams):
        raise RuntimeError("fused streaming kernels (name, bytes of scratch memory per lane): %s" % streams)
    if verbose:
        print("stream kernels checked: %d (compiler writes nothing at or above v80, no calls; %d kernels of the general "
              "epilogue use scratch memory)" % (checked, spilling), flush=True)


def _loops(lines):
    """(first, last) line of every loop: from a label to a branch back to it."""
    import re

    at, found = {}, []
    for i, line in enumerate(lines):
        label, branch = re.match(r"(\.LBB\w+):", line), re.match(r"\s+s_c?branch\w*\s+(\.LBB\w+)", line)
        if label:
            at[label.group(1)] = i
        if branch and branch.group(1) in at:
            found.append((at[branch.group(1)], i))
    return found


def check_int8_attention_loops(verbose: bool = True) -> None:
    """The streaming Int8 attention kernels hold the registers of three to six workgroups on a CU; 96 channels do not quite fit and
    spill a few between the two passes over the keys.  Inside the passes a reload would wait for every direct load on its
    way: this compiles the kernels to assembly and fails if a loop with matrix instructions touches scratch memory."""
    import re

    text, checked = _device_assembly("ogc_mha_i8.hip"), 0
    for m in re.finditer(r"^(_Z24ogc_mha_i8_stream_kernel\w*):[^\n]*\n(.*?)\n\.Lfunc_end", text, re.S | re.M):
        lines = [l.split(";")[0] for l in m.group(2).splitlines()]
        loops = [lines[a:b] for a, b in _loops(lines) if any("v_mfma" in l for l in lines[a:b])]
        if len(loops) < 2:
            raise RuntimeError("%s: the two passes over the keys were not found in the assembly" % m.group(1))
        if any("scratch_" in l for body in loops for l in body):
            raise RuntimeError("%s spills registers in a loop over the keys" % m.group(1))
        checked += 1
    if checked != 4:
        raise RuntimeError("streaming Int8 attention kernels found in the assembly: %d of 4" % checked)
    if verbose:
        print("streaming Int8 attention kernels checked: %d (no spills in the loops over the keys)" % checked, flush=True)


def check_split_attention_loops(verbose: bool = True) -> None:
    """The split fp32 attention kernels use (nearly) all registers, and at 96 channels some are spilled around the loop over the
    keys.  Inside it they must not be: this compiles the kernels to assembly, finds the loop of two rounds (48 matrix instructions
    for 32 channels) and fails if it touches scratch memory more than once (one reload in two rounds is what the masked fast
    softmax at 96 channels has)."""
    import re

    text = _device_assembly("ogc_mha.hip")
    checked = 0
    for m in re.finditer(r"^(_Z14ogc_mha_kernelILi0ELi([123])E\w*):[^\n]*\n(.*?)\n\.Lfunc_end", text, re.S | re.M):
        name, lines, found = m.group(1), [l.split(";")[0] for l in m.group(3).splitlines()], 0
        for first, last in _loops(lines):
            body = lines[first:last]
            if sum("v_mfma_f32_32x32x16_bf16" in l for l in body) != 48 * int(m.group(2)):
                continue
            found += 1
            if sum("scratch_" in l for l in body) > 1:
                raise RuntimeError("%s spills registers in its loop over the keys" % name)
        if not found:
            raise RuntimeError("%s: no loop over the keys found in the assembly" % name)
        checked += 1
    if checked != 12:
        raise RuntimeError("split attention kernels found in the assembly: %d of 12" % checked)
    if verbose:
        print("split attention kernels checked: %d (no spills in the loop over the keys)" % checked, flush=True)


if __name__ == "__main__":
    print(build_library())
    check_stream_kernel_registers()
    check_split_attention_loops()
    check_int8_attention_loops()
    sys.exit(0)
