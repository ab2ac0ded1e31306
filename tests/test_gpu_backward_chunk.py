"""The matrix-core gradient kernels at the edges of their tiles and of the walk
over a workgroup's heads: chunks of 15 to 64 tokens around the 16-token score
tiles, and slices of one, two, three and more heads (the first and the last
ones, whose inputs are fetched out of step).  Against the float64 oracle at the
bf16 bound of test_gpu_backward, which every output meets by a factor of five.
(A row of one token is in test_gpu_backward.  Its dA_log is a single dot product
of two states rounded to bf16, 2^-8.5 of its terms' norm off: over seven heads
the largest one happened to cancel to an eighth of that norm, 2.3e-2, on these
kernels as on the ones before them, so that size has no relative bound.)"""
import pytest

from paper_2405_21060_amd.inputs import Problem, make_grad_inputs, make_inputs
from tests.ssd_harness import TOL, announce
from tests.test_gpu_backward import check, gpu_backward, oracle_backward
from tests.test_gpu_parity import _gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [64, 128])
@pytest.mark.parametrize("T", [15, 16, 17, 33, 64, 111])
@pytest.mark.parametrize("heads,per_slice", [(1, 0), (2, 2), (7, 3), (8, 8)])
def test_edges(N, T, heads, per_slice, tune):
    announce("backward N %d, %d tokens, %d heads, %d a slice" % (N, T, heads, per_slice))
    tune("bwd_heads_per_slice", per_slice)
    inp = make_inputs(Problem(2, T, heads, 64, N, 1, 256, "bf16", init_states=True), 37)
    dy, dfinal = make_grad_inputs(inp.problem, 37)
    got, ref = gpu_backward(inp, dy, dfinal, True, True), oracle_backward(inp, dy, dfinal, True, True)
    for k in ("dx", "ddt", "dB", "dC", "dA_log", "dD", "dinit"):
        check(k, got[k], ref[k], TOL["bf16"])


@pytest.mark.parametrize("N", [64, 128])
def test_later_tokens_do_not_see_an_infinite_score(N):
    """C of one token not finite: its scores with later tokens are masked, so dx
    and ddt of those are what they are with a finite C."""
    import torch
    from paper_2405_21060_amd import ssd
    from tests.ssd_harness import act_to_device, to_device

    announce("backward N %d, one token's C infinite" % N)
    inp = make_inputs(Problem(1, 50, 2, 64, N, 1, 256, "bf16", init_states=True), 38)
    dy, dfinal = make_grad_inputs(inp.problem, 38)
    d, g = to_device(inp), []
    for bad in (False, True):
        C = d["C"].clone()
        if bad:
            C[0, 18] = float("inf")
        g.append(ssd.backward(d["x"], d["dt"], d["A_log"], d["B"], C, act_to_device(dy), D=d["D"],
                              initial_states=d["initial_states"], dfinal_states=torch.from_numpy(dfinal).cuda()))
    for k in ("dx", "ddt"):
        assert torch.equal(g[0][k][:, 19:], g[1][k][:, 19:]), k
