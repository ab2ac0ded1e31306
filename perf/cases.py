"""Timed cases of the SSD layer: what a program that uses this library has it do.

A case names one public entry point of ``paper_2405_21060_amd.ssd`` and the
sizes of one call:

* ``op``      decode, forward, varlen, block, backward, backward_varlen or
              block_backward
* ``dtype``   bf16 or f32 (activations; states and per-head values are float32)
* ``batch``, ``seqlen``, ``heads``, ``headdim``, ``dstate``, ``groups``, ``chunk``
* ``init``    whether the call starts from states (and, for a gradient, whether
              the final states have one)
* ``lengths`` (packed rows) the seed of the sequences' lengths; ``shortest`` and
              ``longest`` bound them; ``host`` whether the boundaries are given
              as host offsets or as the device's ``seq_idx``

Inputs have the distributions of ``paper_2405_21060_amd.inputs``: A in [-16, -1],
dt = softplus(normal + bias) around 1e-3 .. 1e-1, x and dy normal, B and C
normal / sqrt(dstate).
"""
import math
import random

import torch

from paper_2405_21060_amd import ssd

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(op, batch, seqlen, heads, dstate=128, *, name=None, dtype="bf16", headdim=64, groups=1, chunk=256,
          init=False, **more):
    c = {"op": op, "dtype": dtype, "batch": batch, "seqlen": seqlen, "heads": heads, "headdim": headdim,
         "dstate": dstate, "groups": groups, "chunk": chunk, "init": init, **more}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # one new token of one sequence, 24 heads (d_model 768): the smallest call there is
        _case("decode", 1, 1, 24, name="decode_b1"),
        # one new token of each of 256 sequences being served, 80 heads (d_model 2560)
        _case("decode", 256, 1, 80, name="decode_b256"),
        # a prompt of ordinary, odd length, alone in its batch
        _case("forward", 1, 777, 80, name="prefill_t777"),
        # the forward of a training step or of a full prefill batch
        _case("forward", 4, 4096, 80, name="forward_2p7b"),
        # long sequences with the largest state
        _case("forward", 4, 16384, 80, 256, name="forward_t16384_n256"),
        # heads of 128, chunks of 128
        _case("forward", 2, 4096, 40, headdim=128, chunk=128, name="forward_p128"),
        # sequences packed into one row, continued from states, eight groups
        _case("varlen", 1, 32768, 64, groups=8, init=True, lengths=0, shortest=256, longest=4096, host=False,
              name="varlen_g8"),
        # the layer inside its block: dt's softplus in front, gate and RMS norm over the channels behind
        _case("block", 4, 4096, 80, name="block_2p7b"),
        # gradients of a training step's layer, and of a smaller model's block
        _case("backward", 4, 4096, 80, name="backward_2p7b"),
        _case("block_backward", 8, 2048, 24, name="block_backward_130m"),
        # float32 throughout, both directions
        _case("forward", 2, 2048, 24, dtype="f32", name="forward_f32"),
        _case("backward", 2, 2048, 24, dtype="f32", name="backward_f32"),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, even over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _rows(rng, tokens):
    """batch and seqlen of about so many tokens."""
    batch = rng.choice([b for b in (1, 1, 2, 3, 4, 8, 16) if b * 64 <= tokens])
    return batch, max(1, tokens // batch)


def draw(rng):
    op = rng.choice(["decode", "decode", "forward", "forward", "forward", "varlen", "block", "backward", "backward",
                     "backward_varlen", "block_backward", "forward_p128", "forward_f32", "backward_f32"])
    heads = rng.choice([10, 24, 32, 48, 64, 80])
    groups = 8 if heads % 8 == 0 and rng.random() < 0.25 else 1
    dstate = rng.choice([64, 128, 128])
    init = rng.random() < 0.4
    if op == "decode":
        dtype = "f32" if rng.random() < 0.15 else "bf16"
        return _case(op, _log(rng, 1, 256), 1, heads, dstate, dtype=dtype, groups=groups)
    if op == "forward_f32" or op == "backward_f32":
        batch, seqlen = _rows(rng, _log(rng, 100, 4096))
        return _case(op[:-4], batch, seqlen, rng.choice([8, 10, 16, 24]), dstate, dtype="f32",
                     chunk=rng.choice([64, 128, 256]), init=init)
    if op == "forward_p128":
        batch, seqlen = _rows(rng, _log(rng, 100, 8192))
        return _case("forward", batch, seqlen, rng.choice([8, 16, 24, 32, 40]), dstate, headdim=128,
                     chunk=rng.choice([128, 256]), init=init)
    if op in ("varlen", "backward_varlen"):
        shortest, longest = rng.choice([(1, 600), (100, 2000), (256, 4096)])
        return _case(op, 1, _log(rng, 1000, 32768), rng.choice([24, 32, 64]), dstate, groups=groups,
                     init=init, lengths=rng.randrange(1 << 20), shortest=shortest, longest=longest,
                     host=op == "backward_varlen" or rng.random() < 0.5)
    if op == "forward":
        batch, seqlen = _rows(rng, _log(rng, 100, 65536))
        return _case(op, batch, seqlen, heads, rng.choice([64, 128, 128, 256]), groups=groups, init=init)
    batch, seqlen = _rows(rng, _log(rng, 100, 16384))
    return _case(op, batch, seqlen, heads, dstate, groups=groups, init=init)


def _starts(case):
    """Token offsets of a packed row's sequences: lengths between shortest and
    longest until they fill the row, the last one cut."""
    rng = random.Random(case["lengths"])
    starts = [0]
    while starts[-1] < case["seqlen"]:
        starts.append(min(case["seqlen"], starts[-1] + rng.randint(case["shortest"], case["longest"])))
    return starts


def _units(case):
    return len(_starts(case)) - 1 if "lengths" in case else case["batch"]


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype = DTYPES[case["dtype"]]
    b, T, H, P = case["batch"], case["seqlen"], case["heads"], case["headdim"]
    N, G, op = case["dstate"], case["groups"], case["op"]
    row = (b,) if op == "decode" else (b, T)

    def normal(*shape, scale=1.0, kind=dtype):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(scale).to(kind)

    def uniform(lo, hi):
        return torch.rand((H,), generator=gen, device="cuda", dtype=torch.float32).mul_(hi - lo).add_(lo)

    s = {"op": op, "chunk": case["chunk"]}
    s["A_log"] = uniform(0.0, math.log(16.0))
    s["D"] = normal(H, kind=torch.float32)
    s["dt_bias"] = torch.log(torch.expm1(uniform(1e-3, 1e-1)))
    raw = normal(*row, H)
    s["dt"] = raw if op.startswith("block") else torch.nn.functional.softplus(raw.float() + s["dt_bias"]).to(dtype)
    s["x"] = normal(*row, H, P)
    s["B"] = normal(*row, G, N, scale=1 / math.sqrt(N))
    s["C"] = normal(*row, G, N, scale=1 / math.sqrt(N))
    f32 = {"kind": torch.float32}
    units = _units(case)
    s["init"] = normal(units, H, P, N, **f32) if case["init"] or op == "decode" else None
    if op.startswith("block"):
        s["z"] = normal(b, T, H, P)
        s["norm_weight"] = normal(H * P, scale=0.1, **f32).add_(1.0)
        s["norm_group_size"] = H * P // G
    if "backward" in op:
        s["dy"] = normal(b, T, H, P)
        s["dfinal"] = normal(units, H, P, N, **f32) if case["init"] else None
    if "lengths" in case:
        s["starts"] = _starts(case)
        s["nseq"] = units
        ends = torch.tensor(s["starts"][1:], device="cuda")
        s["seq_idx"] = torch.searchsorted(ends, torch.arange(T, device="cuda"), right=True).to(torch.int32).view(1, T)
        s["host"] = case["host"]
    return s


def run(s):
    op = s["op"]
    layer = (s["x"], s["dt"], s["A_log"], s["B"], s["C"])
    if op == "decode":
        return {"y": ssd.decode_step(*layer, s["init"], D=s["D"]), "state": s["init"]}
    if op == "forward":
        y, final = ssd.forward(*layer, D=s["D"], chunk_size=s["chunk"], initial_states=s["init"])
        return {"y": y, "final": final}
    if op == "varlen":
        if s["host"]:
            y, final = ssd.forward_varlen(*layer, s["starts"], D=s["D"], initial_states=s["init"])
        else:
            y, final = ssd.forward(*layer, D=s["D"], initial_states=s["init"], seq_idx=s["seq_idx"], nseq=s["nseq"])
        return {"y": y, "final": final}
    if op == "backward":
        return ssd.backward(*layer, s["dy"], D=s["D"], initial_states=s["init"], dfinal_states=s["dfinal"])
    if op == "backward_varlen":
        return ssd.backward_varlen(*layer, s["dy"], s["starts"], D=s["D"], initial_states=s["init"],
                                   dfinal_states=s["dfinal"])
    block = {k: s[k] for k in ("dt_bias", "z", "norm_weight", "norm_group_size")}
    if op == "block":
        y, final = ssd.forward_block(*layer, D=s["D"], chunk_size=s["chunk"], initial_states=s["init"], **block)
        return {"y": y, "final": final}
    return ssd.backward_block(*layer, s["dy"], D=s["D"], initial_states=s["init"], dfinal_states=s["dfinal"], **block)


def work(case):
    """Each input read once, each output written once, and the operations of the
    recurrence's chunked form on causal pairs (chunks of 64 tokens for a
    gradient, of the call's size for the forward)."""
    b, T, H, P = case["batch"], case["seqlen"], case["heads"], case["headdim"]
    N, G, op = case["dstate"], case["groups"], case["op"]
    tok, size = b * T, 2 if case["dtype"] == "bf16" else 4
    state = 4 * _units(case) * H * P * N
    inputs = size * tok * (H * P + H + 2 * G * N)
    act = size * tok * H * P
    if op == "decode":
        return {"bytes": inputs + act + 2 * state + 8 * H, "flops": 5 * tok * H * P * N}
    if op.startswith("block"):
        inputs += act + 4 * H + 4 * H * P
    if "backward" in op:
        nbytes = 2 * inputs + act + state + (2 * state if case["init"] else 0) + 16 * H
        flops = tok * (64 * G * N + H * (64 * (2 * P + 2 * N) + 10 * P * N))
        return {"bytes": nbytes, "flops": flops}
    Q = case["chunk"]
    nbytes = inputs + act + state * (2 if case["init"] else 1) + 8 * H
    if op == "varlen" and not case["host"]:
        nbytes += 4 * tok
    return {"bytes": nbytes, "flops": tok * ((Q + 1) * N * G + H * ((Q + 1) * P + 4 * N * P))}


def tolerance(case):
    """About four times the error against 64 bits: bf16 rounds results and
    matrix operands (2e-3 to 3e-3); in float32 the rounding of a block's
    cumulative decay exponents shows in the final states (4e-6)."""
    return {"rel": 1.2e-2, "max": 0.15} if case["dtype"] == "bf16" else {"rel": 1.5e-5, "max": 5e-4}


def _layer64(x, dt, A_log, B, C, D, init):
    """The layer on float64 tensors, by blocks of 64 tokens (the sum over a block
    in its quadratic form, the state carried from block to block)."""
    b, T, H, P = x.shape
    G, N = B.shape[2:]
    A = -torch.exp(A_log)
    B, C = (v.repeat_interleave(H // G, 2).transpose(1, 2) for v in (B, C))    # b H T N
    x, a, dt = x.transpose(1, 2), (dt * A).transpose(1, 2), dt.transpose(1, 2)
    state = init if init is not None else x.new_zeros((b, H, P, N))
    out, Q = [], 64
    for t in range(0, T, Q):
        e = min(T, t + Q)
        Bc, Cc, xc = B[:, :, t:e].contiguous(), C[:, :, t:e].contiguous(), x[:, :, t:e].contiguous()
        cs = torch.cumsum(a[:, :, t:e], 2)
        low = torch.ones((e - t, e - t), device=x.device, dtype=torch.bool).tril()
        decay = torch.exp((cs[..., :, None] - cs[..., None, :]).masked_fill(~low, -math.inf))
        u = xc * dt[:, :, t:e, None]
        score = torch.matmul(Cc, Bc.transpose(2, 3).contiguous()) * decay
        y = torch.matmul(score, u) + torch.exp(cs)[..., None] * torch.matmul(Cc, state.transpose(2, 3).contiguous())
        out.append(y + D[:, None, None] * xc)
        left = torch.exp(cs[..., -1:] - cs)[..., None]
        state = torch.exp(cs[..., -1])[..., None, None] * state + torch.matmul(
            (u * left).transpose(2, 3).contiguous(), Bc)
    return torch.cat(out, 2).transpose(1, 2), state


def _gated_norm64(y, z, weight, group):
    g = y * z * torch.sigmoid(z)
    rows = g.reshape(g.shape[0], g.shape[1], -1, group)
    n = rows / torch.sqrt(rows.square().mean(-1, keepdim=True) + 1e-5)
    return (n.reshape(g.shape[0], g.shape[1], -1) * weight).view_as(y)


def exact(case, seed):
    """What ``run`` returns, in 64 bits."""
    s, op = prepare(case, seed), case["op"]
    leaf = {k: s[k].double() for k in ("x", "dt", "A_log", "B", "C", "D", "dt_bias", "init", "z", "norm_weight")
            if s.get(k) is not None}
    if op == "decode":
        dt, H, G = leaf["dt"], case["heads"], case["groups"]
        B, C = (leaf[k].repeat_interleave(H // G, 1) for k in ("B", "C"))
        decay = torch.exp(-dt * torch.exp(leaf["A_log"]))[..., None, None]
        state = decay * leaf["init"] + (dt[..., None] * leaf["x"])[..., None] * B[:, :, None, :]
        return {"y": (state * C[:, :, None, :]).sum(-1) + leaf["D"][:, None] * leaf["x"], "state": state}
    grad = "backward" in op
    if grad:
        for v in leaf.values():
            v.requires_grad_()
        if "init" not in leaf:
            leaf["init"] = torch.zeros((_units(case), case["heads"], case["headdim"], case["dstate"]), device="cuda",
                                       dtype=torch.float64, requires_grad=True)
    with torch.set_grad_enabled(grad):
        dt = leaf["dt"]
        if op.startswith("block"):
            dt = torch.nn.functional.softplus(dt + leaf["dt_bias"])
        layer = (leaf["A_log"], leaf["D"])
        if "lengths" in case:
            ys, finals = [], []
            for k, (lo, hi) in enumerate(zip(s["starts"], s["starts"][1:])):
                y, f = _layer64(leaf["x"][:, lo:hi], dt[:, lo:hi], layer[0], leaf["B"][:, lo:hi], leaf["C"][:, lo:hi],
                                layer[1], leaf["init"][k:k + 1] if "init" in leaf else None)
                ys.append(y)
                finals.append(f)
            y, final = torch.cat(ys, 1), torch.cat(finals, 0)
        else:
            y, final = _layer64(leaf["x"], dt, layer[0], leaf["B"], leaf["C"], layer[1], leaf.get("init"))
        if op.startswith("block"):
            y = _gated_norm64(y, leaf["z"], leaf["norm_weight"], s["norm_group_size"])
        if not grad:
            return {"y": y, "final": final}
        loss = (y * s["dy"].double()).sum()
        if s["dfinal"] is not None:
            loss = loss + (final * s["dfinal"].double()).sum()
        loss.backward()
    names = {"dx": "x", "ddt": "dt", "dB": "B", "dC": "C", "dA_log": "A_log", "dD": "D", "dinit": "init"}
    if op.startswith("block"):
        names.update({"ddt_bias": "dt_bias", "dz": "z", "dnorm_weight": "norm_weight"})
    return {k: leaf[v].grad for k, v in names.items()}
