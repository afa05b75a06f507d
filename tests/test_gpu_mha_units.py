"""The bf16 attention kernel at the edges of its units of 32 keys and of the rule that chooses between its forms (no addend,
addend in LDS, general), against the float64 oracle on the same inputs: within 1e-2, as the other bf16 attention tests."""
import math

import numpy as np
import pytest

from paper_2301_01333_amd import binding, synth
from test_gpu_mha import FAST, STABLE, TOL, as_f64, assert_close, check, heads_view

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seq", [32, 33, 64, 95, 96, 97, 128, 160, 255, 256, 320])
@pytest.mark.parametrize("head_dim", [32, 64, 96, 128])
def test_unit_edges(oracle_mod, seq, head_dim):
    """Whole and ragged units, odd and even numbers of them, one and two query groups, with and without a mask."""
    wl = synth.make_mha("bf16", 2, seq, 2 * head_dim, 2, 7100 + seq + head_dim, name="units S=%d d=%d" % (seq, head_dim))
    check(oracle_mod, wl)
    check(oracle_mod, wl, use_mask=False)
    check(oracle_mod, wl, FAST, use_mask=False)


def run_and_compare(oracle_mod, wl, softmax=STABLE, what=""):
    from paper_2301_01333_amd.harness import DeviceMHA

    dev = DeviceMHA(wl, softmax)
    dev.run()
    q, k, v = (heads_view(as_f64(t), wl) for t in (wl.q, wl.k, wl.v))
    ref = oracle_mod.attention(q, k, v, wl.mask, wl.scale, softmax).transpose(0, 2, 1, 3).reshape(wl.batch, wl.seq, wl.hidden)
    assert_close(as_f64(dev.result()), ref, TOL["bf16"], what or wl.name)
    return dev


@pytest.mark.parametrize("head_dim", [64, 128])
def test_the_reference_of_the_exponentials_moves(oracle_mod, head_dim):
    """Leading units wholly masked, so that the first reference is far below the later scores; then scores that rise by
    hundreds from unit to unit, in either direction; then every key of a row masked alike (a plain mean of the values)."""
    wl = synth.make_mha("bf16", 2, 288, 2 * head_dim, 2, 7300 + head_dim, name="masked prefix")
    wl.mask[:] = 0.0
    wl.mask[:, :70] = -10000.0
    run_and_compare(oracle_mod, wl, what="masked prefix")
    for sign in (1.0, -1.0):
        wl.mask[:] = (sign * 3.0 * np.arange(288, dtype=np.float32))[None]
        run_and_compare(oracle_mod, wl, what="rising mask %g" % sign)
    for level in (-10000.0, -1.0e38):
        wl.mask[:] = 0.0
        wl.mask[1] = level
        run_and_compare(oracle_mod, wl, what="row masked alike at %g" % level)


@pytest.mark.parametrize("scale", [-0.125, 0.0, 1e-33])
def test_scalars_without_a_usable_reciprocal(oracle_mod, scale):
    """The addend cannot be divided by these: the general kernel, with and without a mask."""
    wl = synth.make_mha("bf16", 2, 150, 2 * 64, 2, 7500, name="scale %g" % scale)
    wl.scale = scale
    desc = binding.mha_desc(binding.OGC_BF16, 2, 2, 150, 64, scale)
    assert binding.ogc_mha_kernel_name(desc, True).startswith("ogc_mha_general_kernel<2")
    run_and_compare(oracle_mod, wl)
    run_and_compare(oracle_mod, wl, FAST)


@pytest.mark.parametrize("seq", [4096, 4097, 6200, 8300])
def test_sequences_beyond_the_addends_in_lds(oracle_mod, seq):
    """4096 addends are held at a time; the halves are replaced every 2048 keys (a random mask: every key counts)."""
    wl = synth.make_mha("bf16", 1, seq, 64, 1, 7600 + seq, name="S=%d" % seq)
    wl.mask[:] = np.random.default_rng(seq).standard_normal(wl.mask.shape).astype(np.float32) * 2.0
    run_and_compare(oracle_mod, wl)


def test_token_strides_beyond_32_bits_of_offset(oracle_mod):
    """Keys 64 MiB apart: the general kernel's 64-bit addresses."""
    import torch

    wl = synth.make_mha("bf16", 1, 3, 64, 1, 7700, name="wide token stride")
    ks = (1 << 25) + 8                     # elements between keys: a byte offset of 2^31 / 32 and a little more
    k_dev = torch.zeros(2 * ks + 64, dtype=torch.uint16, device="cuda")
    for i in range(3):
        k_dev[i * ks:i * ks + 64] = torch.from_numpy(wl.k[0, i].copy()).cuda()
    q_dev, v_dev = (torch.from_numpy(t.copy()).cuda() for t in (wl.q, wl.v))
    m_dev = torch.from_numpy(wl.mask.copy()).cuda()
    o_dev = torch.zeros(3 * 64, dtype=torch.uint16, device="cuda")
    desc = binding.mha_desc(binding.OGC_BF16, 1, 1, 3, 64, wl.scale, k_stride=(3 * ks, 64, ks))
    assert binding.ogc_mha_kernel_name(desc, True) == "ogc_mha_general_kernel<2, 0>"
    binding.ogc_mha_run(desc, q_dev.data_ptr(), k_dev.data_ptr(), v_dev.data_ptr(), m_dev.data_ptr(), o_dev.data_ptr(),
                        int(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    q, k, v = (heads_view(as_f64(t), wl) for t in (wl.q, wl.k, wl.v))
    ref = oracle_mod.attention(q, k, v, wl.mask, wl.scale, STABLE).transpose(0, 2, 1, 3).reshape(1, 3, 64)
    assert_close(as_f64(o_dev.cpu().numpy()).reshape(1, 3, 64), ref, TOL["bf16"], "wide token stride")
