"""Normalisation groups around the widths where the block's output pass and its
gradient change kernels: 128 pieces of 8 channels (two a lane of a wavefront),
512 and 1024 (one and two a thread of a workgroup), and past that (with more than
the 512 heads that one pass of d dt holds); rows that do
not fill a chunk of 16.  Against the float64 oracles, at the bounds of
test_gpu_block and test_gpu_block_backward."""
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
