"""The names that ogc_mlp_kernel_name, ogc_mha_kernel_name and ogc_mha_i8_kernel_name report are those of kernels in the library
(host only: names and symbols are compared, nothing runs)."""
import itertools
import os
import re
import shutil
import subprocess

import pytest

from paper_2301_01333_amd import binding as b

pytestmark = pytest.mark.skipif(not os.path.exists(b.LIB_PATH), reason="libogc_mlp.so not built (python -m paper_2301_01333_amd.build)")


@pytest.fixture(scope="module")
def kernels():
    nm = shutil.which("nm") or "/opt/rocm/llvm/bin/llvm-nm"
    out = subprocess.run([nm, "-C", "--defined-only", b.LIB_PATH], check=True, capture_output=True, text=True).stdout
    names = set(re.findall(r"\bvoid (ogc_\w+<[^>]*>)\(", out))
    assert "ogc_layer_dma_kernel<2, 0, 1, 0, 1>" in names
    return names


def chain(dtype, dims, **more):
    quant = dict(in_scale=0.05, in_zp=128 if dtype == b.OGC_I8 else 0, out_scale=0.1, out_zp=128 if dtype == b.OGC_I8 else 0)
    return [dict(dict(k=k, n=n, has_bias=1, act=b.OGC_ACT_RELU, out=0, **quant), **more) for k, n in zip(dims, dims[1:])]


def chain_name(dtype, m, dims, mode, overrides=None, ld_x=None, **more):
    """The names of all layers of a plan; none if the plan is refused."""
    try:
        p = b.ogc_mlp_plan_with_overrides(dtype, m, chain(dtype, dims, **more), ld_x or dims[0], dims[-1], 0, mode, overrides=overrides)
    except b.OgcError:
        return set()
    names = {b.ogc_mlp_kernel_name(p, l) for l in range(len(dims) - 1)}
    b.ogc_mlp_destroy(p)
    return names


@pytest.mark.parametrize("dtype", [b.OGC_F32, b.OGC_BF16, b.OGC_I8, b.OGC_F8])
def test_every_reported_chain_kernel_is_in_the_library(kernels, dtype):
    forced = [{"tile": t} for t in range(6)] + [{"tile": t, "ksplit_log2": 1} for t in (3, 4, 5)]
    forced += [{"cluster_split": s, "cluster_ksplit": k} for s in (0, 2, 4, 8) for k in (0, 1)]
    for m, dims in itertools.product((1, 256, 8192, 9000), ([64, 64, 64], [37, 130, 9], [479, 1024, 1024, 512, 256, 1], [1024, 1024, 1024])):
        reported = set()
        for mode, ov in itertools.product((b.OGC_MODE_AUTO, b.OGC_MODE_PER_LAYER, b.OGC_MODE_FUSED, b.OGC_MODE_COOP), [None] + forced):
            for act in (b.OGC_ACT_RELU, b.OGC_ACT_GELU_TANH, b.OGC_ACT_NONE):
                reported |= chain_name(dtype, m, dims, mode, ov, act=act)
        assert reported and reported <= kernels, reported - kernels


def test_every_reported_attention_kernel_is_in_the_library(kernels):
    for dtype, d, seq, batch in itertools.product((b.OGC_F32, b.OGC_BF16, b.OGC_I8), (32, 64, 96, 128), (1, 33, 64, 200, 512), (1, 64)):
        for softmax, mask, groups in itertools.product((b.OGC_SOFTMAX_STABLE, b.OGC_SOFTMAX_FAST), (True, False), (0, 1, 2)):
            desc = b.mha_desc(dtype, batch, 4, seq, d, 0.1, softmax)
            desc.query_groups = groups
            name = b.ogc_mha_i8_kernel_name(desc) if dtype == b.OGC_I8 else b.ogc_mha_kernel_name(desc, mask)
            assert not name or name in kernels, name


@pytest.mark.parametrize("dtype, width, ld_x, name", [
    (b.OGC_BF16, 64, 64, "rows_chain_kernel<1>"), (b.OGC_BF16, 64, 72, "rows_chain_kernel<1>"), (b.OGC_BF16, 64, 68, "chain_kernel<1>"),
    (b.OGC_BF16, 60, 64, "chain_kernel<1>"), (b.OGC_F8, 64, 64, "rows_chain_kernel<3>"), (b.OGC_F8, 64, 72, "chain_kernel<3>"),
    (b.OGC_I8, 64, 64, "chain_kernel<2>"), (b.OGC_F32, 64, 64, "chain_kernel<0>")])
def test_cluster_kernel_name_tells_how_rows_are_staged(dtype, width, ld_x, name):
    """bf16 and E4M3 rows on 16-byte boundaries have a kernel of their own."""
    ov = {"cluster_split": 2, "cluster_ksplit": 0}
    assert chain_name(dtype, 100, [width, 96, 64], b.OGC_MODE_COOP, ov, ld_x) == {"ogc_cluster_" + name}


@pytest.mark.parametrize("dtype, m, dims, name", [
    # a megabyte (1000000 bytes) of packed weights, inner widths padded to 32 channels (bf16) or 64
    (b.OGC_I8, 256, [1024, 960, 32], "stream_kernel<2>"), (b.OGC_I8, 256, [1024, 896, 32], "kernel<2>"), (b.OGC_BF16, 100, [512, 992], "stream_kernel<1>"),
    (b.OGC_BF16, 100, [512, 960], "kernel<1>"), (b.OGC_F8, 100, [1000, 1000], "stream_kernel<3>"), (b.OGC_F8, 100, [960, 1024], "kernel<3>"),
    (b.OGC_F32, 100, [512, 512], "kernel<0>"),
    # at most a sixth of them in layers of fewer than eight k-steps
    (b.OGC_I8, 100, [192, 1024, 1024], "stream_kernel<2>"), (b.OGC_I8, 100, [192, 1280, 960], "stream_kernel<2>"), (b.OGC_I8, 100, [192, 1280, 928], "kernel<2>"),
    (b.OGC_BF16, 1, [96, 640, 800], "stream_kernel<1>"), (b.OGC_I8, 100, [1000, 130, 1000, 1000], "stream_kernel<2>"), (b.OGC_I8, 100, [100, 1500, 100, 1500, 700], "kernel<2>"),
    # beyond 256 row tiles, where LDS holds two workgroups, the pair kernel comes first
    (b.OGC_I8, 8192, [1024, 1024, 1024], "stream_kernel<2>"), (b.OGC_F8, 8193, [1024, 1024, 1024], "pair_kernel<3>")])
def test_fused_kernel_name_tells_the_stream(kernels, dtype, m, dims, name):
    """Which chains have their weights streamed across blocks and layers."""
    assert chain_name(dtype, m, dims, b.OGC_MODE_FUSED) == {"ogc_fused_chain_" + name}
    assert "ogc_fused_chain_" + name in kernels
