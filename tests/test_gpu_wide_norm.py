"""Normalisation groups around the widths where the block's output pass and its
gradient change kernels: 128 pieces of 8 channels (two a lane of a wavefront),
512 and 1024 (one and two a thread of a workgroup), and past that (with more than
the 512 heads that one pass of d dt holds); rows that do
not fill a chunk of 16.  Against the float64 oracles, at the bounds of
test_gpu_block and test_gpu_block_backward."""
import numpy as np
import pytest

import oracle.block as ob
from paper_2405_21060_amd.inputs import Problem, make_block_inputs, make_grad_inputs
from tests.ssd_harness import TOL, announce, rel_err, to_f64
from tests.test_gpu_block import run_block
from tests.test_gpu_block_backward import BASE, check, run_gpu, run_oracle
from tests.test_gpu_parity import _gpu  # noqa: F401

pytestmark = pytest.mark.gpu

# heads, headdim, groups, channels per normalisation group
SHAPES = [(64, 16, 1, 1024), (65, 16, 1, 1040), (130, 16, 2, 1040), (64, 64, 1, 4096), (65, 64, 1, 4160),
          (128, 64, 1, 8192), (513, 16, 1, 8208)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("gate,weight", [(True, True), (False, False)])
@pytest.mark.parametrize("H,P,G,group", SHAPES)
def test_wide_groups(H, P, G, group, gate, weight, dtype):
    announce("norm group %d of %d channels %s gate %s weight %s" % (group, H * P, dtype, gate, weight))
    p = Problem(1, 37, H, P, 64, G, 256, dtype)
    bi = make_block_inputs(p, 41)
    opts = dict(gate=gate, norm_group_size=group, norm_weight=weight)
    y, fin = run_block(bi, opts)
    y_ref, fin_ref = ob.block_forward_inputs(bi, opts)
    assert rel_err(to_f64(y), y_ref) <= TOL[dtype]
    assert rel_err(to_f64(fin), fin_ref) <= TOL[dtype]

    o = dict(BASE, gate=gate, weight=weight, group=group, dt_raw=bi.dt_raw)
    dout, _ = make_grad_inputs(p, 41)
    got, ref = run_gpu(bi, dout, None, o), run_oracle(bi, dout, None, o)
    for k in ("dx", "dA_log", "dB", "dC", "ddt_bias") + (("dz",) if gate else ()) + (("dnorm_weight",) if weight else ()):
        check(k, got[k], ref[k], TOL[dtype])
    check("ddt_raw", got["ddt"], ref["ddt_raw"], TOL[dtype])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("gate,weight", [(True, True), (False, False)])
@pytest.mark.parametrize("rows,H,P,G,group", [
    (8, 65, 64, 1, 4160), (9, 65, 64, 1, 4160),          # one chunk: few rows, too many
    (240, 65, 16, 1, 1040), (241, 65, 16, 1, 1040),      # 15 and 16 workgroups
    (1264, 65, 16, 1, 1040), (1265, 65, 16, 1, 1040),    # 79 and 80
    (640, 130, 16, 2, 1040)])                            # 40 chunks of two groups
def test_row_counts(rows, H, P, G, group, gate, weight, dtype):
    """Rows on both sides of the lines where the gradient's kernels change."""
    announce("norm group %d, %d rows %s gate %s weight %s" % (group, rows, dtype, gate, weight))
    p = Problem(1, rows, H, P, 64, G, 256, dtype)
    bi = make_block_inputs(p, 43)
    o = dict(BASE, gate=gate, weight=weight, group=group, dt_raw=bi.dt_raw)
    dout, _ = make_grad_inputs(p, 43)
    got, ref = run_gpu(bi, dout, None, o), run_oracle(bi, dout, None, o)
    for k in ("dx", "dA_log", "dB", "dC", "ddt_bias") + (("dz",) if gate else ()) + (("dnorm_weight",) if weight else ()):
        check(k, got[k], ref[k], TOL[dtype])
    check("ddt_raw", got["ddt"], ref["ddt_raw"], TOL[dtype])


@pytest.mark.parametrize("heads", [33, 80])
def test_gate_is_exact_to_float32(heads):
    """The gate's SiLU, seen through a rounding of the result to bf16: y is x (B =
    C = 0, D = 1), gated by z and normalised over the row, and each channel's
    weight puts the exact result 1e-6 of its value above or below the middle of
    two bf16 values.  Float32's errors (SiLU 2e-7, the weight and three products
    2^-24 each, the root 2^-23, and none in the mean square, which is far below
    eps) add up to 6e-7: every channel has to land on its side."""
    import torch
    from paper_2405_21060_amd import ssd
    from paper_2405_21060_amd.inputs import bf16_bits_to_f32, f32_to_bf16_bits

    announce("gate to float32, %d heads" % heads)
    rng = np.random.default_rng(45)
    n = heads * 64
    z = np.concatenate([rng.uniform(-85.0, -20.0, n - n // 8), rng.uniform(-88.5, -85.0, n // 8)])
    z = bf16_bits_to_f32(f32_to_bf16_bits(rng.permutation(z).astype(np.float32))).astype(np.float64)
    x = rng.choice([-1.0, -2.0, 0.5, 4.0], n)
    k, side = rng.integers(0, 127, n), rng.choice([-1, 1], n)
    mid = 1.0 + (2 * k + 1) / 256.0
    g = x * z / (1.0 + np.exp(-z))
    w = (mid * (1.0 + 1e-6 * side) / (g / np.sqrt((g * g).mean() + 1e-5))).astype(np.float32)
    dev = lambda a, *s: torch.from_numpy(a).cuda().to(torch.bfloat16).view(1, 1, *s)
    zero = torch.zeros((1, 1, 1, 64), dtype=torch.bfloat16, device="cuda")
    one = torch.ones(heads, device="cuda")
    y, _ = ssd.forward_block(dev(x, heads, 64), torch.zeros((1, 1, heads), dtype=torch.bfloat16, device="cuda"), one,
                             zero, zero, one, z=dev(z, heads, 64), norm_weight=torch.from_numpy(w).cuda(),
                             norm_group_size=n)
    wrong = np.flatnonzero(to_f64(y).reshape(-1) != mid + side / 256.0)
    assert wrong.size == 0, (wrong.size, z[wrong[:8]], to_f64(y).reshape(-1)[wrong[:8]], mid[wrong[:8]], side[wrong[:8]])
