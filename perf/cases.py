"""The measured workloads of libm3: the calls that programs built on it make.

Each case is one call of a public entry point, over the shapes that the
package's workload table, tests and benchmark use, plus ragged lengths:

* decode: `step` / `step_pro`, from one sequence (latency) to a serving batch;
* prefill: `scan_fwd` (plain, gated, per-head frequencies, continued from a
  state and carry), `scan_fwd_pro` (the Mamba-3 block with its norm, biases,
  structured input, gate and output norm), `scan_fwd_varlen` (packed batch);
* training: `scan_bwd`.

Inputs follow the package's synthetic distributions (inputs.py).  A program
keeps its workspace and its output buffers between calls where the entry
point takes them, so they are made in `prepare`.
"""
from __future__ import annotations

import ctypes
import math
import random

import torch

from paper_2603_15569_amd import inputs, m3, roofline

IO = {"f32": torch.float32, "bf16": torch.bfloat16}


# --------------------------------------------------------------------------
# Cases
# --------------------------------------------------------------------------

def _scan(name, batch, seqlen, nheads, rank, chunk, io="bf16", headdim=64, dstate=128,
          gate=False, theta="token", init=False):
    return dict(name=name, kind="scan", batch=batch, seqlen=seqlen, nheads=nheads, rank=rank,
                chunk=chunk, io=io, headdim=headdim, dstate=dstate, gate=gate, theta=theta,
                init=init)


def _block(name, batch, seqlen, nheads, rank, chunk, onorm=2):
    return dict(name=name, kind="block", batch=batch, seqlen=seqlen, nheads=nheads, rank=rank,
                chunk=chunk, io="bf16", headdim=64, dstate=128, gate=True, theta="token",
                init=False, onorm=onorm)


def _varlen(name, nseq, shortest, longest, nheads, rank, chunk, lens_seed, theta="token"):
    return dict(name=name, kind="varlen", nseq=nseq, shortest=shortest, longest=longest,
                nheads=nheads, rank=rank, chunk=chunk, io="bf16", headdim=64, dstate=128,
                gate=False, theta=theta, init=False, lens_seed=lens_seed)


def _bwd(name, batch, seqlen, nheads, rank, a="head"):
    return dict(name=name, kind="bwd", batch=batch, seqlen=seqlen, nheads=nheads, rank=rank,
                chunk=64 // rank, io="bf16", headdim=64, dstate=128, a=a)


def _step(name, batch, nheads, rank, io="bf16", headdim=64, dstate=128, block=False,
          theta="token"):
    return dict(name=name, kind="step", batch=batch, nheads=nheads, rank=rank, io=io,
                headdim=headdim, dstate=dstate, block=block, theta=theta)


def listed():
    return [
        # one token of one sequence in an interactive session: launch latency
        _step("decode_one", 1, 32, 1),
        # a mid-size serving batch through the whole block (norms, biases, gate)
        _step("decode_block", 24, 32, 4, block=True),
        # the serving batch of the decode benchmark
        _step("decode_batch", 256, 32, 4),
        # the small fp32 scan that the fp32 build serves
        _scan("prefill_tiny_fp32", 1, 256, 2, 1, 64, io="f32", headdim=16, dstate=16),
        # SISO layer over a small training or prefill batch
        _scan("prefill_siso", 4, 2048, 16, 1, 64),
        # rank-4 layer over a full batch
        _scan("prefill_mimo", 8, 4096, 32, 4, 64),
        # one long document
        _scan("prefill_long", 1, 65536, 32, 4, 128),
        # the Mamba-3 block on a couple of prompts of odd length
        _block("prefill_block", 2, 4001, 32, 4, 64),
        # the smaller state of the paper's sweep, gated, a prompt continued
        _scan("prefill_state64", 4, 2000, 16, 1, 64, dstate=64, gate=True, init=True),
        # prompts of mixed lengths packed into one call
        _varlen("prefill_packed", 24, 17, 2000, 16, 2, 64, 7, theta="head"),
        # a training step's backward: SISO, and the rank-4 layer at full batch
        _bwd("backward_siso", 4, 2048, 16, 1),
        _bwd("backward_mimo", 8, 4096, 32, 4),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _split(rng, rows, rank, min_len, max_len):
    """Batch, length and heads of about `rows` (token, head, rank) rows."""
    nheads = rng.choice([2, 4, 8, 12, 16, 24, 32, 48])
    nheads = max(1, min(nheads, rows // (rank * min_len)))
    tokens = max(min_len, rows // (rank * nheads))
    longest = max(min_len, min(max_len, tokens))
    seqlen = _log_int(rng, min(longest, max(min_len, tokens // 512)), longest)
    return max(1, tokens // seqlen), seqlen, nheads


_CHUNKS = {1: (64, 128), 2: (32, 64, 128), 4: (32, 64, 128)}


def draw(rng):
    kind = rng.choice(["step", "scan", "scan", "block", "varlen", "small", "fp32", "bwd", "bwd"])
    rank = rng.choice([1, 2, 4])
    theta = rng.choice(["token", "token", "head"])
    if kind == "step":
        io, headdim, dstate = rng.choice([("bf16", 64, 128), ("bf16", 64, 128), ("bf16", 64, 64),
                                          ("bf16", 64, 32), ("f32", 64, 128), ("f32", 16, 16)])
        block = io == "bf16" and dstate == 128 and rng.random() < 0.5
        c = _step("", _log_int(rng, 1, 256), rng.choice([4, 8, 16, 24, 32]), rank, io, headdim,
                  dstate, block, theta)
    elif kind == "scan":
        b, n, h = _split(rng, _log_int(rng, 1 << 12, 1 << 22), rank, 33, 65536)
        c = _scan("", b, n, h, rank, rng.choice(_CHUNKS[rank]), gate=rng.random() < 0.5,
                  theta=theta, init=rng.random() < 0.5)
    elif kind == "block":
        b, n, h = _split(rng, _log_int(rng, 1 << 12, 1 << 22), rank, 33, 65536)
        c = _block("", b, n, h, rank, rng.choice(_CHUNKS[rank]), rng.choice([0, 1, 2]))
    elif kind == "varlen":
        longest = _log_int(rng, 64, 4096)
        nseq = _log_int(rng, 2, max(2, min(256, (1 << 16) // longest)))
        c = _varlen("", nseq, 1, longest, rng.choice([4, 8, 16]), rank,
                    rng.choice(_CHUNKS[rank]), rng.randrange(1 << 30), theta)
    elif kind == "small":
        dstate = rng.choice([64, 64, 32])
        chunk = rng.choice({64: {1: (64, 128), 2: (32, 64), 4: (16, 32)},
                            32: {1: (64,), 2: (32,), 4: (16,)}}[dstate][rank])
        b, n, h = _split(rng, _log_int(rng, 1 << 12, 1 << 20), rank, 33, 16384)
        c = _scan("", b, n, h, rank, chunk, dstate=dstate, gate=rng.random() < 0.5, theta=theta,
                  init=rng.random() < 0.5)
    elif kind == "fp32":
        headdim, dstate = rng.choice([(64, 128), (16, 16)])
        chunk = rng.choice({16: {1: (64,), 2: (32, 64), 4: (16, 32, 64)},
                            128: {1: (32,), 2: (32,), 4: (16, 32)}}[dstate][rank])
        if dstate == 128 and rank == 1:
            rank = 2
        b, n, h = _split(rng, _log_int(rng, 1 << 10, 1 << 18), rank, 33, 16384)
        c = _scan("", b, n, h, rank, chunk, io="f32", headdim=headdim, dstate=dstate, theta=theta,
                  init=rng.random() < 0.5)
    else:
        b, n, h = _split(rng, _log_int(rng, 1 << 12, 3 << 20), rank, 33, 16384)
        # (a decay per head for layers of several heads: its gradient is one
        # number a head, a sum over every token that can cancel)
        c = _bwd("", b, n, h, rank, rng.choice(["head", "token"]) if h >= 8 else "token")
    del c["name"]
    return c


# --------------------------------------------------------------------------
# What a program holds before the call
# --------------------------------------------------------------------------

def _lengths(case):
    """Sequence lengths of a packed batch: over the logarithm of the range."""
    rng = random.Random(case["lens_seed"])
    return [_log_int(rng, case["shortest"], case["longest"]) for _ in range(case["nseq"])]


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(0x5EED + int(seed))
    return g


def _randn(g, *shape):
    return torch.randn(shape, device="cuda", generator=g)


def _rms(v):
    return v * torch.rsqrt(v.pow(2).mean(dim=-1, keepdim=True) + 1e-6)


def _state_like(case, batch, inp, g):
    """A state and carry as a sequence in progress has them: entries at the
    steady state's scale of each head."""
    H, N, P, R, io = case["nheads"], case["dstate"], case["headdim"], case["rank"], IO[case["io"]]
    dt = torch.nn.functional.softplus(inp.dt_bias)
    decay = 1.0 - torch.exp(2.0 * dt * inp.A)
    scale = dt * torch.sqrt(R / decay)
    state = _randn(g, batch, H, N, P) * scale[None, :, None, None]
    cB = _rms(_randn(g, batch, H, R, N)).to(io)
    cX = _randn(g, batch, H, R, P).to(io)
    return state, cB, cX


def _pro_tables(case, pi, onorm, og):
    return dict(bc_norm=True, eps=1e-6, norm_B=pi.gB, norm_C=pi.gC, bias_B=pi.bB, bias_C=pi.bC,
                w_x=pi.wx, w_z=pi.wz, out_norm=onorm, out_group=case["headdim"] if onorm else 0,
                out_gain=og if onorm else None)


def _outputs(batch, case, like):
    H, N, P, R = case["nheads"], case["dstate"], case["headdim"], case["rank"]
    return (torch.empty_like(like), torch.empty(batch, H, N, P, device="cuda"),
            torch.empty(batch, H, R, N, device="cuda", dtype=like.dtype),
            torch.empty(batch, H, R, P, device="cuda", dtype=like.dtype))


def _inputs(case, seed):
    """The tensors of a case, from the seed alone."""
    g = _generator(seed)
    H, N, P, R = case["nheads"], case["dstate"], case["headdim"], case["rank"]
    kind = case["kind"]
    if kind == "step":
        b = case["batch"]
        layer = inputs.make_scan_inputs(b, 1, H, P, N, R, io=case["io"], seed=seed, device="cuda")
        t = dict(x=layer.x[:, 0], Bm=layer.Bm[:, 0], Cm=layer.Cm[:, 0], dt=layer.dt[:, 0],
                 lam=layer.lam[:, 0], theta=layer.theta[:, 0], A=layer.A, D=layer.D)
        if case["theta"] == "head":
            t["theta"] = layer.omega
        t["state"], t["cB"], t["cX"] = _state_like(case, b, layer, g)
        if case["block"]:
            pi = inputs.make_prologue_inputs(b, 1, H, P, N, R, io=case["io"], seed=seed,
                                             device="cuda")
            t["x"], t["z"], t["Bm"], t["Cm"] = pi.xp[:, 0], pi.zp[:, 0], pi.Bp[:, 0], pi.Cp[:, 0]
            t["tables"] = _pro_tables(case, pi, 2, 0.5 + torch.rand(H, R, P, device="cuda", generator=g))
        return {k: v.contiguous() if isinstance(v, torch.Tensor) else v for k, v in t.items()}
    if kind == "varlen":
        lens = _lengths(case)
        batch, seqlen = 1, sum(lens)
    else:
        batch, seqlen = case["batch"], case["seqlen"]
    inp = inputs.make_scan_inputs(batch, seqlen, H, P, N, R, io=case["io"], seed=seed,
                                  device="cuda")
    t = dict(x=inp.x, Bm=inp.Bm, Cm=inp.Cm, dt=inp.dt, A=inp.A, lam=inp.lam, theta=inp.theta,
             D=inp.D)
    if kind == "bwd":
        t["dy"] = _randn(g, *inp.x.shape).to(inp.x.dtype)
        if case["a"] == "token":   # the data-dependent decay of the Mamba-3 layer
            t["A"] = inp.A * torch.exp(0.25 * _randn(g, batch, seqlen, H))
        return t
    if case["theta"] == "head":
        t["theta"] = inp.omega
    if case["init"]:
        t["state"], t["cB"], t["cX"] = _state_like(case, batch, inp, g)
    if kind == "block":
        del t["x"], t["Bm"], t["Cm"], inp
        pi = inputs.make_prologue_inputs(batch, seqlen, H, P, N, R, io=case["io"], seed=seed,
                                         device="cuda")
        t["x"], t["z"], t["Bm"], t["Cm"] = pi.xp, pi.zp, pi.Bp, pi.Cp
        t["tables"] = _pro_tables(case, pi, case["onorm"], 0.5 + torch.rand(H, R, P, device="cuda", generator=g))
    elif case["gate"]:
        t["z"] = _randn(g, *inp.x.shape).to(inp.x.dtype)
    if kind == "varlen":
        cu = [0]
        for n in lens:
            cu.append(cu[-1] + n)
        t["cu"] = cu
        for k in ("x", "Bm", "Cm", "dt", "lam") + (("theta",) if case["theta"] == "token" else ()):
            t[k] = t[k][0]
    return t


def prepare(case, seed):
    t = _inputs(case, seed)
    kind, Q = case["kind"], case.get("chunk")
    st = dict(kind=kind, t=t, chunk=Q, rank=case["rank"])
    args = (t["x"], t["Bm"], t["Cm"], t["dt"], t["A"], t["lam"], t["theta"], t["D"])
    st["args"] = args
    if kind == "step":
        st["pro"] = m3.prologue(**t["tables"]) if case["block"] else None
        st["y"] = torch.empty(case["batch"], case["nheads"], case["rank"], case["headdim"],
                              device="cuda", dtype=IO[case["io"]])
        return st
    st["init"] = dict(init_state=t["state"], init_carry=(t["cB"], t["cX"])) if case.get("init") else {}
    ph = case.get("theta") == "head"
    if kind == "scan":
        d = m3.scan_dims(t["x"], t["Bm"], Q, t["A"], theta_per_head=ph)
        st["ws"] = torch.zeros(max(m3.workspace_bytes(d), 16), dtype=torch.uint8, device="cuda")
        st["out"] = _outputs(case["batch"], case, t["x"])
    elif kind == "block":
        st["pro"] = m3.prologue(**t["tables"])
        b, n, h, r, p = case["batch"], case["seqlen"], case["nheads"], case["rank"], case["headdim"]
        y = torch.empty(b, n, h, r, p, device="cuda", dtype=IO[case["io"]])
        d = m3.scan_dims(y, t["Bm"], Q, t["A"], theta_per_head=ph)
        st["ws"] = torch.zeros(max(m3.workspace_bytes(d), 16), dtype=torch.uint8, device="cuda")
        st["out"] = _outputs(b, case, y)
    elif kind == "varlen":
        d = m3.varlen_dims(t["x"], t["Bm"], t["A"], Q, t["cu"], theta=t["theta"])
        one = m3.varlen_workspace_bytes(d, t["cu"])
        st["ws"] = torch.zeros(one, dtype=torch.uint8, device="cuda") if one else None
    else:
        d = m3.scan_dims(t["x"], t["Bm"], Q, t["A"])
        n = int(m3.lib().m3_scan_bwd_workspace_bytes(ctypes.byref(d)))
        st["ws"] = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    return st


# --------------------------------------------------------------------------
# One pass
# --------------------------------------------------------------------------

def run(st):
    t, kind = st["t"], st["kind"]
    if kind == "step":
        carry = (t["cB"], t["cX"])
        if st["pro"] is None:
            y = m3.step(t["state"], carry, *st["args"], y=st["y"])
        else:
            y = m3.step_pro(t["state"], carry, *st["args"], st["pro"], z=t["z"], y=st["y"])
        return {"y": y, "state": t["state"], "cB": t["cB"], "cX": t["cX"]}
    if kind == "bwd":
        return m3.scan_bwd(*st["args"], t["dy"], st["chunk"], workspace=st["ws"])
    if kind == "scan":
        y, fs, (cB, cX) = m3.scan_fwd(*st["args"], chunk=st["chunk"], out=st["out"],
                                      workspace=st["ws"], z=t.get("z"), **st["init"])
    elif kind == "block":
        y, fs, (cB, cX) = m3.scan_fwd_pro(*st["args"], chunk=st["chunk"], pro=st["pro"],
                                          rank=st["rank"], z=t["z"], out=st["out"],
                                          workspace=st["ws"], **st["init"])
    else:
        y, fs, (cB, cX) = m3.scan_fwd_varlen(*st["args"], chunk=st["chunk"], cu_seqlens=t["cu"],
                                             workspace=st["ws"], z=t.get("z"), **st["init"])
    return {"y": y, "state": fs, "cB": cB, "cX": cX}


# --------------------------------------------------------------------------
# Algorithmic work, tolerances
# --------------------------------------------------------------------------

def work(case):
    H, N, P, R = case["nheads"], case["dstate"], case["headdim"], case["rank"]
    io = 4 if case["io"] == "f32" else 2
    kind = case["kind"]
    ph = case.get("theta") == "head"
    if kind == "step":
        b = case["batch"]
        per = roofline.decode_bytes_per_slice(N, P, R, io) - (2 * N if ph else 0)
        if case["block"]:   # X', Z' of P values in place of x
            per += (2 * P - R * P) * io
        return {"bytes": b * H * per, "flops": b * H * roofline.decode_flops_per_slice(N, P, R)}
    if kind == "bwd":
        b, n = case["batch"], case["seqlen"]
        return {"bytes": roofline.backward_bytes(b, n, H, N, P, R, io),
                "flops": b * H * roofline.backward_flops(n, N, P, R, case["chunk"])}
    if kind == "varlen":
        n, b = sum(_lengths(case)), 1
    else:
        b, n = case["batch"], case["seqlen"]
    nbytes = roofline.prefill_bytes(b, n, H, N, P, R, io)
    if kind == "varlen":
        nbytes += (case["nseq"] - 1) * H * (N * P * 4 + R * (N + P) * io)
    if ph:
        nbytes -= b * n * H * 2 * N
    if case["init"]:
        nbytes += b * H * (N * P * 4 + R * (N + P) * io)
    if kind == "block":
        nbytes += b * n * H * (2 * P - R * P) * io
    elif case["gate"]:
        nbytes += b * n * H * R * P * io
    return {"bytes": nbytes, "flops": b * H * roofline.chunked_flops(n, N, P, R, case["chunk"])}


def tolerance(case):
    if case["io"] == "f32":
        # fp32 products and sums, fp64 angle and decay prefixes: 1e-7 to 3e-7
        # from the 64-bit result as the sums' lengths and order vary
        return {"rel": 1e-5}
    if case["kind"] == "step":
        # fp32 update, hardware sine, cosine and exponential, bf16 outputs (1.7e-3
        # from the 64-bit result), bf16 B and C after the block's norm (2.8e-3)
        return {"rel": 1e-2}
    if case["kind"] == "bwd":
        # bf16 operands and gradients (2.4e-3 to 4.1e-3), and per head the sum of
        # dA over every token, of both signs (2e-3 to 7e-3)
        return {"rel": 2.5e-2}
    # bf16 operands, scores and outputs (2.3e-3 to 3.7e-3 from the 64-bit result)
    return {"rel": 1.5e-2}


# --------------------------------------------------------------------------
# The same in 64 bits: the recurrence's masked form in chunks, in the frame
# that rotates with the cumulative angle of the whole sequence
# --------------------------------------------------------------------------

def _rotate(v, psi, sign):
    """Rotate the pairs (i, i + N/2) of v [b, L, R, N] by sign * psi [b, L, N/2]."""
    c, s = torch.cos(psi).unsqueeze(2), sign * torch.sin(psi).unsqueeze(2)
    re, im = v.chunk(2, dim=-1)
    return torch.cat([c * re - s * im, s * re + c * im], dim=-1)


def _head64(x, B, C, dt, dA, lam, theta, D, h0=None, cB=None, cX=None, Q=32):
    """One head in float64: x [b,L,R,P], B and C [b,L,R,N], dt, dA = dt A and
    lam [b,L], theta [b,L,N/2] angles.  Returns y and the final state."""
    b, L, R, P = x.shape
    N = B.shape[-1]
    psi = torch.cumsum(theta, 1)
    Bh, Ch = _rotate(B, psi, -1.0), _rotate(C, psi, -1.0)
    gam = lam * dt
    sig = gam + torch.nn.functional.pad(((1 - lam) * dt)[:, 1:], (0, 1))
    n = -(-L // Q)
    pad = n * Q - L

    def chunks(v, *shape):
        v = torch.nn.functional.pad(v, (0, 0) * (v.dim() - 2) + (0, pad))
        return v.reshape(b, n, *shape)

    xc = chunks(x, Q * R, P)
    Bc, Cc = chunks(Bh, Q * R, N), chunks(Ch, Q * R, N)
    cum = torch.cumsum(chunks(dA, Q), 2)
    gc, sc = chunks(gam, Q), chunks(sig, Q)
    tot = cum[:, :, -1]
    low = torch.tril(torch.ones(Q, Q, dtype=torch.bool, device=x.device), -1)
    diff = (cum[..., :, None] - cum[..., None, :]).masked_fill(~low, 0.0)
    w = torch.where(low, torch.exp(diff) * sc[..., None, :], torch.diag_embed(gc))
    w = w.repeat_interleave(R, -1).repeat_interleave(R, -2)
    y = torch.matmul(torch.matmul(Cc, Bc.transpose(-1, -2).contiguous()) * w, xc)
    v = (torch.exp(tot[..., None] - cum) * sc).repeat_interleave(R, -1)
    M = torch.matmul((Bc * v[..., None]).transpose(-1, -2).contiguous(), xc)      # [b, n, N, P]
    # chunk states: S_c = e^{tot_c} S_{c-1} + M_c, unrolled over blocks of chunks
    s = torch.zeros(b, N, P, dtype=x.dtype, device=x.device) if h0 is None else h0
    if cB is not None:
        s = s + ((1 - lam[:, 0]) * dt[:, 0])[:, None, None] * torch.matmul(cB.transpose(-1, -2).contiguous(), cX)
    states = []
    for k0 in range(0, n, 64):
        m = min(64, n - k0)
        t = torch.cumsum(tot[:, k0:k0 + m], 1)
        tri = torch.tril(torch.ones(m, m, dtype=torch.bool, device=x.device))
        f = torch.where(tri, torch.exp((t[:, :, None] - t[:, None, :]).masked_fill(~tri, 0.0)), 0.0)
        out = torch.matmul(f, M[:, k0:k0 + m].reshape(b, m, N * P)).reshape(b, m, N, P)
        out = out + torch.exp(t)[..., None, None] * s[:, None]
        states.append(torch.cat([s[:, None], out[:, :-1]], 1))
        s = out[:, -1]
    S = torch.cat(states, 1)
    e = torch.exp(cum).repeat_interleave(R, -1)
    y = y + e[..., None] * torch.matmul(Cc, S)
    y = y.reshape(b, n * Q, R, P)[:, :L] + D * x
    fs = _rotate(s.transpose(1, 2).unsqueeze(1), psi[:, -1:], 1.0).squeeze(1).transpose(1, 2)
    return y, fs


def _silu(z):
    return z * torch.sigmoid(z)


def _prologue64(t, h, Bm, Cm, x, z):
    """Norm, gains and biases of B and C and the structured input and gate,
    of head h (any leading axes, then [R,N] or [P])."""
    tb = t["tables"]

    def norm(v, gain, bias):
        v = v * torch.rsqrt(v.pow(2).mean(-1, keepdim=True) + tb["eps"])
        return v * gain[h].double() + bias[h].double()

    Bm, Cm = norm(Bm, tb["norm_B"], tb["bias_B"]), norm(Cm, tb["norm_C"], tb["bias_C"])
    return Bm, Cm, x.unsqueeze(-2) * tb["w_x"][h].double(), z.unsqueeze(-2) * tb["w_z"][h].double()


def _epilogue64(t, h, y, z):
    """Output norm (before or after the gate) over whole rows, and the gate."""
    tb = t["tables"]
    if tb["out_norm"] == 2:
        y = y * _silu(z)
    if tb["out_norm"]:
        y = y * torch.rsqrt(y.pow(2).mean(-1, keepdim=True) + 1e-6) * tb["out_gain"][h].double()
    return y if tb["out_norm"] == 2 else y * _silu(z)


def _angles(t, h, dt):
    th = t["theta"]
    if th.dim() == 2:   # frequencies: the angle is dt * omega
        return dt.unsqueeze(-1) * th[h].double()
    return th[..., h, :].double()


def exact(case, seed):
    t = _inputs(case, seed)
    kind, H = case["kind"], case["nheads"]
    f = lambda name, h: t[name][..., h, :, :].double()          # noqa: E731
    if kind == "step":
        R, N, P, b = case["rank"], case["dstate"], case["headdim"], case["batch"]
        y = torch.empty(b, H, R, P, dtype=torch.float64, device="cuda")
        state, cB, cX = t["state"].double(), t["cB"].double(), t["cX"].double()
        for h in range(H):
            B, C, dt, lam = f("Bm", h), f("Cm", h), t["dt"][:, h].double(), t["lam"][:, h].double()
            if case["block"]:
                B, C, x, z = _prologue64(t, h, B, C, t["x"][:, h].double(), t["z"][:, h].double())
            else:
                x = f("x", h)
            yh, fs = _head64(x[:, None], B[:, None], C[:, None], dt[:, None],
                             (dt * t["A"][h].double())[:, None], lam[:, None],
                             _angles(t, h, dt)[:, None], t["D"][h].double(), state[:, h], cB[:, h],
                             cX[:, h], Q=1)
            y[:, h] = _epilogue64(t, h, yh[:, 0], z) if case["block"] else yh[:, 0]
            state[:, h], cB[:, h], cX[:, h] = fs, B, x
        return {"y": y, "state": state, "cB": cB, "cX": cX}
    if kind == "bwd":
        return _exact_bwd(case, t)
    if kind == "varlen":
        parts = []
        for a, z in zip(t["cu"], t["cu"][1:]):
            one = dict(t)
            for k in ("x", "Bm", "Cm", "dt", "lam") + (("theta",) if t["theta"].dim() == 3 else ()):
                one[k] = t[k][a:z].unsqueeze(0)
            parts.append(_exact_scan(case, one))
        return {k: torch.cat([p[k][0] if k == "y" else p[k] for p in parts]) for k in parts[0]}
    return _exact_scan(case, t)


def _exact_scan(case, t):
    f = lambda name, h: t[name][..., h, :, :].double()          # noqa: E731
    H, N, P, R = case["nheads"], case["dstate"], case["headdim"], case["rank"]
    b, L = t["dt"].shape[:2]
    new = lambda *s: torch.empty(*s, dtype=torch.float64, device="cuda")   # noqa: E731
    out = {"y": new(b, L, H, R, P), "state": new(b, H, N, P), "cB": new(b, H, R, N), "cX": new(b, H, R, P)}
    for h in range(H):
        B, C, dt, lam = f("Bm", h), f("Cm", h), t["dt"][..., h].double(), t["lam"][..., h].double()
        z = None
        if case["kind"] == "block":
            B, C, x, z = _prologue64(t, h, B, C, t["x"][..., h, :].double(), t["z"][..., h, :].double())
        else:
            x = f("x", h)
            if case["gate"]:
                z = f("z", h)
        init = (t["state"][:, h].double(), t["cB"][:, h].double(), t["cX"][:, h].double()) if case["init"] else ()
        y, fs = _head64(x, B, C, dt, dt * t["A"][h].double(), lam, _angles(t, h, dt),
                        t["D"][h].double(), *init)
        if case["kind"] == "block":
            y = _epilogue64(t, h, y, z)
        elif z is not None:
            y = y * _silu(z)
        out["y"][:, :, h], out["state"][:, h], out["cB"][:, h], out["cX"][:, h] = y, fs, B[:, -1], x[:, -1]
    return out


def _exact_bwd(case, t):
    """Gradients by automatic differentiation of the float64 form, head by head."""
    H, N, P, R = case["nheads"], case["dstate"], case["headdim"], case["rank"]
    b, L = t["dt"].shape[:2]
    new = lambda *s: torch.empty(*s, dtype=torch.float64, device="cuda")   # noqa: E731
    token = t["A"].dim() == 3
    out = {"dx": new(b, L, H, R, P), "dB": new(b, L, H, R, N), "dC": new(b, L, H, R, N),
           "ddt": new(b, L, H), "dlam": new(b, L, H), "dtheta": new(b, L, H, N // 2),
           "dD": new(H), "dA": new(b, L, H) if token else new(H)}
    for h in range(H):
        v = [t[k][:, :, h].double().requires_grad_() for k in ("x", "Bm", "Cm", "dt", "lam", "theta")]
        A = (t["A"][..., h] if token else t["A"][h]).double().requires_grad_()
        D = t["D"][h].double().requires_grad_()
        x, B, C, dt, lam, theta = v
        y, _ = _head64(x, B, C, dt, dt * A, lam, theta, D, Q=max(1, 64 // R))
        grads = torch.autograd.grad(y, [*v, A, D], t["dy"][:, :, h].double())
        for k, g in zip(("dx", "dB", "dC", "ddt", "dlam", "dtheta"), grads):
            out[k][:, :, h] = g
        if token:
            out["dA"][:, :, h] = grads[6]
        else:
            out["dA"][h] = grads[6]
        out["dD"][h] = grads[7]
    return out
