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


@pytest.mark.parametrize("shape", [(64, 128, 1, "f32"), (80, 144, 2, "f32"), (128, 64, 1, "bf16"), (16, 16, 1, "f32")], ids=str)
@pytest.mark.parametrize("name,token", [("dy", 18), ("dy", 70), ("C", 18), ("C", 64), ("B", 27), ("B", 95)])
def test_an_infinite_operand_stays_with_its_pairs(shape, name, token):
    """One token's dy, C or B infinite: the gradients whose sums leave that token
    out are what they are without it -- dx and ddt of later tokens for dy, dB of
    later tokens for C, dC of earlier ones for B -- although its score tile holds
    their (zero) scores too.  (Up to the order of a tile's float32 sum: 2^-24
    times its sixteen terms, relative to the largest gradient.)"""
    import numpy as np
    import torch
    from paper_2405_21060_amd import ssd
    from tests.ssd_harness import act_to_device, to_device, to_f64

    P, N, G, dtype = shape
    announce("general backward P%d N%d %s, %s of token %d infinite" % (P, N, dtype, name, token))
    inp = make_inputs(Problem(1, 100, 4, P, N, G, 256, dtype, init_states=True), 33)
    dy, dfinal = make_grad_inputs(inp.problem, 33)
    d = to_device(inp)
    d["dy"] = act_to_device(dy)
    g = []
    for bad in (False, True):
        t = {k: d[k].clone() for k in ("dy", "C", "B")}
        if bad:
            t[name][0, token] = float("inf")
        g.append(ssd.backward(d["x"], d["dt"], d["A_log"], t["B"], t["C"], t["dy"], D=d["D"],
                              initial_states=d["initial_states"], dfinal_states=torch.from_numpy(dfinal).cuda()))
    far = slice(0, token) if name == "B" else slice(token + 1, None)
    for k in {"dy": ("dx", "ddt"), "C": ("dB",), "B": ("dC",)}[name]:
        a, b = to_f64(g[0][k])[:, far], to_f64(g[1][k])[:, far]
        assert np.all(np.isfinite(b)), k
        assert np.abs(a - b).max() <= (2.0 ** -20 if dtype == "f32" else 2.0 ** -8) * np.abs(a).max(), k
