"""The general backward kernels at the edges of their tiles: 16-token score
tiles and 64-token chunks, feature and column blocks of 64, one and several
head slices, float32 and bf16.  Against the float64 oracle, at the bounds of
test_gpu_backward; float32 also at 2e-5 (sums over at most a few thousand terms
in float32, whose rounding grows as their square root: 1e-7 x 60, times three)."""
import pytest

from paper_2405_21060_amd.inputs import Problem, make_grad_inputs, make_inputs
from tests.ssd_harness import TOL, announce
from tests.test_gpu_backward import check, gpu_backward, oracle_backward
from tests.test_gpu_parity import _gpu  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [
    # b, T, H, P, N, G
    (1, 64, 2, 64, 128, 1), (2, 65, 3, 64, 64, 1), (1, 63, 2, 80, 144, 2), (1, 17, 4, 112, 16, 2),
    (2, 129, 2, 128, 192, 1), (1, 48, 3, 96, 256, 3), (1, 1, 1, 48, 80, 1), (1, 200, 7, 16, 96, 1),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("per_slice", [0, 2])
def test_edges(shape, dtype, per_slice, tune):
    announce("general backward %s %s, %d heads a slice" % (shape, dtype, per_slice))
    tune("force_general_path", 1)
    tune("bwd_heads_per_slice", per_slice)
    b, T, H, P, N, G = shape
    inp = make_inputs(Problem(b, T, H, P, N, G, 256, dtype, init_states=True), 31)
    dy, dfinal = make_grad_inputs(inp.problem, 31)
    got, ref = gpu_backward(inp, dy, dfinal, True, True), oracle_backward(inp, dy, dfinal, True, True)
    for k in ("dx", "ddt", "dB", "dC", "dA_log", "dD", "dinit"):
        check(k, got[k], ref[k], TOL[dtype])
        if dtype == "f32":
            check(k, got[k], ref[k], 2e-5)


def test_decay_that_vanishes(tune):
    """A underflowed to zero (a head that never forgets) and a head that forgets
    within a token: finite gradients, those of the oracle."""
    announce("general backward, A = 0 and A = -e^6")
    inp = make_inputs(Problem(1, 100, 4, 64, 64, 1, 256, "f32", init_states=True), 32)
    inp.A_log[0], inp.A_log[1] = -200.0, 6.0
    dy, dfinal = make_grad_inputs(inp.problem, 32)
    got, ref = gpu_backward(inp, dy, dfinal, True, True), oracle_backward(inp, dy, dfinal, True, True)
    for k in ("dx", "ddt", "dB", "dC", "dA_log", "dD", "dinit"):
        check(k, got[k], ref[k], 2e-5)
