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


@pytest.mark.parametrize("N", [64, 128])
def test_decays_below_the_normal_range(N):
    """A decay of 2^-130 is a float32 value (19 bits of it) and counts as one: a
    state of 1e30 decayed by it gives dC of order 1e-9.  dC_0 = exp(dt A) h^T dy_0
    with x = 0, each element a sum over 64 features of products of bf16 values
    (the state is one), rounded to bf16."""
    import torch
    from paper_2405_21060_amd import ssd

    announce("backward N %d, decay 2^-130" % N)
    gen = torch.Generator().manual_seed(39)
    bf = lambda *s: torch.randn(s, generator=gen).bfloat16()
    H = 2
    x, B, C = torch.zeros(1, 1, H, 64).bfloat16(), bf(1, 1, 1, N), bf(1, 1, 1, N)
    dt, A_log = torch.ones(1, 1, H).bfloat16(), torch.full((H,), 90.1).log()
    dy, init = bf(1, 1, H, 64), (torch.randn((1, H, 64, N), generator=gen) * 1e30).bfloat16().float()
    g = ssd.backward(*(t.cuda() for t in (x, dt, A_log, B, C, dy)), initial_states=init.cuda())
    decay = torch.exp(-A_log.double().exp())
    terms = decay[:, None, None] * dy[0, 0].double()[:, :, None] * init[0].double()
    ref = terms.sum((0, 1))
    # half a bf16 unit of the value, and float32's exponent (2^-24 of 130, over
    # log2 e) and the decay's own rounding (2^-20) on the terms' sum
    bound = 2.0 ** -8 * ref.abs() + 2.0 ** -16 * terms.abs().sum((0, 1))
    assert ref.abs().min() > 0
    assert bool(((g["dC"].cpu().double()[0, 0, 0] - ref).abs() <= bound).all())
