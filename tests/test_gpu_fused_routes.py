"""Calls that the fused kernels take over from the general ones: headdim 128
(two of their heads a head) and block lengths other than their own, plain and
packed rows, with the block steps -- and the calls of those shapes that stay on
the general kernels (operands off 16 bytes, a workspace of the general size,
packed rows of short sequences, more rows than the fused grid).
Against the float64 oracle, at the bounds of test_gpu_parity, and, for which
kernels ran, against the forced general path bit for bit.
"""
import numpy as np
import pytest

import oracle
import oracle.block as ob
from paper_2405_21060_amd.inputs import Problem, make_block_inputs, make_inputs
from tests.ssd_harness import TOL, announce, rel_err, run_gpu, to_device, to_f64
from tests.test_gpu_block import run_block
from tests.test_gpu_parity import _gpu, compare  # noqa: F401

pytestmark = pytest.mark.gpu

PLAIN = [
    # b, T, H, P, N, G, Q
    (2, 300, 3, 128, 64, 1, 128),      # odd heads, two chunks, the last one partial
    (1, 513, 4, 128, 128, 2, 256),
    (1, 270, 2, 128, 256, 2, 32),      # one head a group, two column blocks
    (3, 1, 5, 128, 128, 1, 64),        # one token
    (2, 257, 6, 64, 128, 3, 32),
    (1, 600, 8, 64, 64, 1, 64),
    (1, 255, 4, 64, 256, 1, 128),
]


def _inputs(b, T, H, P, N, G, Q, seed, **kw):
    return make_inputs(Problem(b, T, H, P, N, G, Q, "bf16", init_states=True, **kw), seed)


def _same_as_general(tune, outputs, call):
    """Whether `outputs` are bit for bit the general kernels' (the two sum in
    different orders, so that only the same kernels give the same bits)."""
    import torch

    tune("force_general_path", 1)
    general = call()
    tune("force_general_path", 0)
    return all(torch.equal(a, b) for a, b in zip(outputs, general))


@pytest.mark.parametrize("shape", PLAIN)
def test_plain_rows(shape, tune):
    announce("fused route %s" % (shape,))
    inp = _inputs(*shape, seed=11)
    y, fin = run_gpu(inp)
    compare(inp, y, fin)
    assert not _same_as_general(tune, (y, fin), lambda: run_gpu(inp))
    y, fin = run_gpu(inp, use_D=False, use_init=False)
    inp.D, inp.initial_states = np.zeros_like(inp.D), None
    compare(inp, y, fin)


@pytest.mark.parametrize("P,N,G,Q", [(128, 128, 1, 256), (128, 64, 2, 64), (64, 128, 2, 128)])
@pytest.mark.parametrize("host", [False, True])
def test_packed_rows(P, N, G, Q, host, tune):
    from paper_2405_21060_amd import ssd

    announce("fused route, packed P%d N%d G%d Q%d host %s" % (P, N, G, Q, host))
    inp = _inputs(1, 1500, 4, P, N, G, Q, seed=12, varlen=True, len_lo=1, len_hi=600)
    if not host:
        y, fin = run_gpu(inp)
        compare(inp, y, fin)
        assert not _same_as_general(tune, (y, fin), lambda: run_gpu(inp))
        return
    d = to_device(inp)
    starts = [0] + [int(v) + 1 for v in np.flatnonzero(np.diff(inp.seq_idx[0]))] + [1500]
    call = lambda: ssd.forward_varlen(d["x"], d["dt"], d["A_log"], d["B"], d["C"], starts, d["D"], chunk_size=Q,
                                      initial_states=d["initial_states"])
    y, fin = call()
    compare(inp, y, fin)
    assert not _same_as_general(tune, (y, fin), call)


@pytest.mark.parametrize("P,Q", [(128, 256), (64, 64)])
@pytest.mark.parametrize("length,general", [(16, True), (32, False)])
def test_short_packed_sequences_stay_general(tune, P, Q, length, general):
    """A chunk per sequence costs the fused kernels 256 tokens' work: rows of
    sequences shorter than 24 tokens on average run on the general kernels."""
    announce("packed, sequences of %d, P%d Q%d" % (length, P, Q))
    inp = _inputs(1, 500, 3, P, 128, 1, Q, seed=20, varlen=True, len_lo=length, len_hi=length)
    y, fin = run_gpu(inp)
    compare(inp, y, fin)
    assert _same_as_general(tune, (y, fin), lambda: run_gpu(inp)) == general


@pytest.mark.parametrize("group", [0, 128, 512])
def test_block_headdim_128(group, tune):
    announce("fused route, block P128 norm group %d" % group)
    bi = make_block_inputs(Problem(2, 400, 4, 128, 128, 2, 128, "bf16"), 13)
    opts = dict(norm_group_size=group)
    y, fin = run_block(bi, opts)
    y_ref, fin_ref = ob.block_forward_inputs(bi, opts)
    assert rel_err(to_f64(y), y_ref) <= TOL["bf16"]
    assert rel_err(to_f64(fin), fin_ref) <= TOL["bf16"]
    assert not _same_as_general(tune, (y, fin), lambda: run_block(bi, opts))


@pytest.mark.parametrize("what", ["x", "B", "C", "y"])
def test_operand_off_16_bytes_stays_general(what, tune):
    """An activation one element off: the general kernels' result, as before."""
    import torch
    from paper_2405_21060_amd import ssd

    announce("general kernels, %s off 16 bytes" % what)
    inp = _inputs(1, 300, 4, 128, 64, 2, 128, seed=14)
    d = to_device(inp)

    def off(t):
        u = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)[1:].view(t.shape)
        return u.copy_(t)

    out = torch.empty_like(d["x"])
    if what == "y":
        out = off(out)
    else:
        d[what] = off(d[what])
    call = lambda: ssd.forward(d["x"], d["dt"], d["A_log"], d["B"], d["C"], d["D"], chunk_size=128,
                               initial_states=d["initial_states"], out=out)
    y, fin = call()
    compare(inp, y, fin)
    y = y.clone()
    assert _same_as_general(tune, (y, fin), call)


def test_workspace_of_the_general_size_is_enough(tune):
    """A one-chunk call whose ring is larger than the general kernels' states."""
    import torch
    from paper_2405_21060_amd import ssd

    announce("general kernels on their own workspace")
    inp = _inputs(2, 32, 16, 128, 128, 1, 32, seed=15)
    d = to_device(inp)
    p = ssd.make_problem(2, 32, 16, 128, 128, 1, 32, ssd.SSD_DTYPE_BF16)
    best = ssd.ssd_workspace_bytes(p)
    tune("force_general_path", 1)
    general = ssd.ssd_workspace_bytes(p)
    tune("force_general_path", 0)
    assert general < best
    y, fin = torch.empty_like(d["x"]), torch.empty_like(d["initial_states"])
    for size, want in ((general, ssd.SSD_OK), (general - 1, ssd.SSD_ERR_WORKSPACE)):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        rc = ssd.ssd_forward(p, *(d[k].data_ptr() for k in ("x", "dt", "A_log", "B", "C", "D", "initial_states")), 0,
                             y.data_ptr(), fin.data_ptr(), ws.data_ptr(), size,
                             torch.cuda.current_stream().cuda_stream)
        assert rc == want
    torch.cuda.synchronize()
    compare(inp, y, fin)
    assert _same_as_general(tune, (y, fin), lambda: run_gpu(inp))


@pytest.mark.parametrize("P,Q,N,packed", [(128, 256, 128, False), (128, 64, 64, True), (64, 128, 128, False),
                                          (64, 32, 256, True)])
def test_scores_are_rounded_once(P, Q, N, packed):
    """The Gram matrix of these shapes is float32: a score C_t . B_s times its
    decay and dt_s is rounded to bf16 once, as a matrix operand.  With x = 1 at
    one token of a chunk and zero at the others (no skip term, no state), y_t is
    that one operand exactly, so its error is at most half a unit in the last
    place, 2^-8 of the value (and 2^-13 for the decay's float32 exponent and the
    sum over N, whose terms have one sign).  Rounded twice it comes near 2^-7."""
    from paper_2405_21060_amd.inputs import f32_to_bf16_bits

    announce("one rounding, P%d Q%d N%d packed %s" % (P, Q, N, packed))
    T = 512 if packed else 256
    inp = make_inputs(Problem(1 if packed else 2, T, 3, P, N, 1, Q, "bf16", varlen=packed, len_lo=256, len_hi=256), 16)
    rng = np.random.default_rng(17)
    inp.A_log[:] = rng.uniform(-1.0, 0.0, 3)
    inp.dt[:] = f32_to_bf16_bits(rng.uniform(0.01, 0.05, inp.dt.shape))
    inp.B[:] = inp.B & 0x7FFF
    inp.C[:] = inp.C & 0x7FFF
    inp.x[:] = 0
    inp.x[:, 0::256] = 0x3F80   # one token of each chunk
    y, _ = run_gpu(inp, use_D=False)
    inp.D = np.zeros_like(inp.D)
    ref, _ = oracle.forward_inputs(inp)
    assert ref.min() > 0
    assert (np.abs(to_f64(y) - ref) / ref).max() <= 2.0 ** -8 + 2.0 ** -13


@pytest.mark.parametrize("P,N", [(128, 128), (128, 256), (128, 64)])
def test_final_states_round_the_weighted_x(P, N):
    """The rounded operand of the state update at these shapes is x_s dt_s
    exp(cs_end - cs_s).  Against that sum in float64 the final states differ
    where the float32 weight (relative error about 2^-20) lands on the other
    side of a rounding: a share of 2^-20 / 2^-8 of the operands, by 2^-8 of
    their value, so 2^-14 of the norm, and the sum's own float32 rounding; four
    times that is asked for.  Another operand rounded gives 2e-3."""
    from paper_2405_21060_amd.inputs import bf16_bits_to_f32, f32_to_bf16_bits

    announce("weighted x, P%d N%d" % (P, N))
    inp = make_inputs(Problem(2, 250, 3, P, N, 1, 256, "bf16"), 18)
    inp.A_log[:] = np.random.default_rng(19).uniform(-1.0, 0.0, 3)
    _, fin = run_gpu(inp)
    x, dt, B = (inp.as_f64(k) for k in ("x", "dt", "B"))
    cs = np.cumsum(dt * -np.exp(inp.A_log.astype(np.float64)), 1)
    xw = (x * (dt * np.exp(cs[:, -1:] - cs))[..., None]).astype(np.float32)
    xw = bf16_bits_to_f32(f32_to_bf16_bits(xw)).astype(np.float64)
    ref = np.matmul(xw.transpose(0, 2, 3, 1), B[:, :, 0][:, None])
    assert np.linalg.norm(to_f64(fin) - ref) <= 4 * 2.0 ** -14 * np.linalg.norm(ref)


@pytest.mark.parametrize("host", [False, True])
def test_python_callers_workspace_of_the_general_size(tune, host):
    """``forward`` and ``forward_varlen`` hand a caller's workspace on as it is:
    the general kernels' size is enough, one byte less is refused."""
    import torch
    from paper_2405_21060_amd import ssd

    announce("general kernels on a Python caller's workspace, host offsets %s" % host)
    inp = _inputs(1, 64, 8, 128, 128, 1, 32, seed=21, varlen=True, len_lo=32, len_hi=32)
    d, starts = to_device(inp), [0, 32, 64]
    p = ssd.make_problem(1, 64, 8, 128, 128, 1, 32, ssd.SSD_DTYPE_BF16, 2)
    size = lambda: ssd.ssd_forward_varlen_workspace_bytes(p, starts) if host else ssd.ssd_workspace_bytes(p)
    best = size()
    tune("force_general_path", 1)
    general = size()
    tune("force_general_path", 0)
    assert general < best

    def call(ws):
        args = (d["x"], d["dt"], d["A_log"], d["B"], d["C"])
        kw = dict(chunk_size=32, initial_states=d["initial_states"], workspace=ws)
        if host:
            return ssd.forward_varlen(*args, starts, d["D"], **kw)
        return ssd.forward(*args, d["D"], seq_idx=d["seq_idx"], nseq=2, **kw)

    compare(inp, *call(torch.empty(general, dtype=torch.uint8, device="cuda")))
    with pytest.raises(ValueError):
        call(torch.empty(general - 1, dtype=torch.uint8, device="cuda"))


def test_more_rows_than_the_fused_grid():
    """66,000 batch rows x groups: past the fused kernels' grid, on the general ones."""
    announce("general kernels, 33,000 rows of two groups")
    inp = make_inputs(Problem(33000, 1, 2, 128, 64, 2, 32, "bf16"), 22)
    y, _ = run_gpu(inp, final=False)
    compare(inp, y, None)


@pytest.mark.parametrize("P,Q", [(128, 256), (64, 128)])
def test_decays_below_the_normal_range(P, Q):
    """A decay of 2^-130 counts as one: with x of 1e30 at the first token, zero
    elsewhere, and scores of 2^17 (their products with the decay are in the
    normal range again), y of the tokens a step later is that operand, rounded to
    bf16 once, times 1e30, rounded again: 2^-7 in all, and 2^-16 for the decay's
    own 19 bits and float32's exponent."""
    import torch
    from paper_2405_21060_amd import ssd

    announce("fused route, decay 2^-130, P%d Q%d" % (P, Q))
    T, H, N = 40, 2, 128
    gen = torch.Generator().manual_seed(23)
    B = (32.0 * (1.0 + torch.rand((1, T, 1, N), generator=gen))).bfloat16()
    C = (32.0 * (1.0 + torch.rand((1, T, 1, N), generator=gen))).bfloat16()
    x = torch.zeros(1, T, H, P).bfloat16()
    x[:, 0] = 1e30
    dt = torch.zeros(1, T, H).bfloat16()
    dt[:, 0], dt[:, 20] = 1.0, 1.0   # the decay falls between the tokens 19 and 20
    A_log = torch.full((H,), 90.1).log()
    y, _ = ssd.forward(x.cuda(), dt.cuda(), A_log.cuda(), B.cuda(), C.cuda(), chunk_size=Q)
    decay = torch.exp(-A_log.double().exp())[None, :] ** (torch.arange(T) >= 20)[:, None]
    ref = (C[0, :, 0].double() @ B[0, 0, 0].double())[:, None] * decay * x[0, 0, 0, 0].double()
    err = ((y[0].cpu().double() - ref[..., None]).abs() / ref[..., None]).max()
    assert err <= 2.0 ** -7 + 2.0 ** -16


@pytest.mark.parametrize("early", [1, 2])
@pytest.mark.parametrize("heads", [1, 2, 4])
@pytest.mark.parametrize("P,N,packed", [(128, 64, False), (128, 128, True), (64, 256, False), (128, 256, True),
                                        (64, 128, False)])
def test_kernel_variants(tune, P, N, packed, heads, early):
    """Late and early state flag, one and several heads an item, several items a
    workgroup (their Gram tiles and operands fetched ahead)."""
    announce("fused route P%d N%d packed %s, %d heads an item, flag %d" % (P, N, packed, heads, early))
    tune("early_state_flag", early)
    tune("heads_per_item", heads)
    tune("max_workgroups", 3)
    inp = _inputs(1 if packed else 2, 900, 4, P, N, 1, 256 if P == 128 else 64, seed=24,
                  **(dict(varlen=True, len_lo=100, len_hi=600) if packed else {}))
    y, fin = run_gpu(inp)
    compare(inp, y, fin)
    assert not _same_as_general(tune, (y, fin), lambda: run_gpu(inp))
