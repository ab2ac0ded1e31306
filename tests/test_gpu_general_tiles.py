"""The general kernels at the edges of their tiles: 16-token strips, 64-token
slabs, 64 x 64 state tiles (features x columns), every chunk length, float32
and bf16, with activations that are aligned to their own type only.  Against
the float64 oracle, at the bounds of test_gpu_parity; float32 also at 2e-5,
about four times the rounding of a chunk's cumulative decay exponents (float32
sums of up to 256 terms, exponents up to some hundred: 1e-7 x 100 / 2)."""
import numpy as np
import pytest

import oracle
from paper_2405_21060_amd.inputs import Problem, make_inputs
from tests.ssd_harness import announce, rel_err, to_device, to_f64
from tests.test_gpu_parity import _gpu, compare  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [
    # b, T, H, P, N, G, Q
    (1, 256, 2, 64, 128, 1, 256), (2, 257, 2, 64, 64, 2, 256), (1, 65, 3, 80, 80, 1, 128),
    (1, 63, 2, 48, 144, 1, 64), (1, 511, 2, 112, 16, 2, 256), (1, 47, 2, 96, 256, 1, 32),
    (2, 17, 4, 128, 192, 4, 64), (1, 1, 2, 16, 16, 1, 32), (1, 1100, 1, 32, 48, 1, 64),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_edges(shape, dtype, tune):
    import torch
    from paper_2405_21060_amd import ssd

    announce("general tiles %s %s" % (shape, dtype))
    tune("force_general_path", 1)
    inp = make_inputs(Problem(*shape, dtype, init_states=True), 21)
    d = to_device(inp)
    for shift in (0, 1):   # as allocated, then one element off
        def put(t):
            u = torch.empty(t.numel() + shift, dtype=t.dtype, device=t.device)[shift:].view(t.shape)
            return u.copy_(t)
        y, fin = ssd.forward(put(d["x"]), put(d["dt"]), d["A_log"], put(d["B"]), put(d["C"]), d["D"],
                             chunk_size=shape[-1], initial_states=put(d["initial_states"]), out=put(d["x"]),
                             final_out=put(d["initial_states"]))
        compare(inp, y, fin)
        if dtype == "f32":
            y_ref, fin_ref = oracle.forward_inputs(inp)
            assert rel_err(to_f64(y), y_ref) <= 2e-5 and rel_err(to_f64(fin), fin_ref) <= 2e-5


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_packed_edges(dtype, tune):
    """Sequences that end on, before and after strip, slab and chunk edges."""
    tune("force_general_path", 1)
    from tests.ssd_harness import run_gpu

    announce("general tiles, packed %s" % dtype)
    lens = [16, 15, 1, 32, 64, 63, 65, 1, 1, 128, 127, 129, 200]
    T = sum(lens)
    inp = make_inputs(Problem(1, T, 3, 80, 96, 3, 128, dtype, varlen=True, init_states=True), 22)
    inp.seq_idx = np.repeat(np.arange(len(lens), dtype=np.int32), lens).reshape(1, T)
    inp.nseq = len(lens)
    inp.initial_states = np.random.default_rng(2).standard_normal((len(lens), 3, 80, 96)).astype(np.float32)
    compare(inp, *run_gpu(inp))
