"""Performance cases of the Float8 library, through the entry points that a training program calls.

Four kinds of case:
  linear     one Float8 linear, forward and backward (f8.linear_fwd / linear_bwd and their delayed-scaling forms),
             or a forward alone against weight codes that the program keeps (f8.linear_fwd_wq).
  attention  the middle of a transformer block: rotary embedding of q and k, causal grouped-query attention, and
             their backward, from the fused q|k|v tensor to its gradient.
  glue       the bf16 operations between the linears: RMSNorm and the SiLU gate, forward and backward.
  block      one whole transformer block (block.TransformerBlock), forward and backward.

Sizes are those of workloads.py (Llama-3.1 linears, one 8B block), of the tests, or generic.  All inputs are drawn
on the GPU from the seed.
"""
import math

import torch

from paper_2410_06511_amd import f8
from paper_2410_06511_amd.block import TransformerBlock

EPS = 1e-5
THETA = 500000.0
HD = 128
HISTORY = 16
FMAX = {f8.E4M3: 448.0, f8.E5M2: 57344.0}
F8_TYPE = {f8.E4M3: torch.float8_e4m3fn, f8.E5M2: torch.float8_e5m2}


# ---- the cases ----------------------------------------------------------------------------

def _linear(name, M, K, N, scaling="dynamic", rowwise=False, e5m2=False, step=True):
    return dict(name=name, kind="linear", M=M, K=K, N=N, scaling=scaling, rowwise=rowwise, e5m2=e5m2, step=step)


def listed():
    return [
        # the smallest configuration of the benchmark: a few microseconds of arithmetic, so launches and latency count
        _linear("linear_256x512x1024", 256, 512, 1024),
        # a short micro-batch against weights whose codes are kept between optimizer steps: the weight's bytes are
        # what the product has to move
        _linear("forward_kept_weight_64", 64, 4096, 4096, step=False),
        # wk / wv of the 8B model at one sequence of 8192 tokens: a narrow output, few tiles in its weight gradient
        _linear("linear_8b_wk", 8192, 4096, 1024),
        # w1 / w3 of the 8B model at two sequences: the largest linear that a training step of it has
        _linear("linear_8b_w1", 16384, 4096, 14336),
        # packed sequences rarely fill a round number of tokens: 2000 = 16 x 125; gradients in e5m2
        _linear("linear_ragged_tokens", 2000, 4096, 4096, e5m2=True),
        # wq of the 405B model split over eight devices, one scale per row and column
        _linear("linear_405b_wq_rowwise", 8192, 16384, 2048, rowwise=True),
        # w2 of the 70B model split over eight devices under delayed scaling, gradients in e5m2
        _linear("linear_70b_w2_delayed", 8192, 3584, 8192, scaling="delayed", e5m2=True),
        # the attention of the 8B model on one sequence of 8192 tokens
        dict(name="attention_8b", kind="attention", B=1, S=8192, Hq=32, Hkv=8),
        # several shorter sequences of a length that no tile divides, every query head with its own keys
        dict(name="attention_4x1000", kind="attention", B=4, S=1000, Hq=16, Hkv=16),
        # norms and gate of the 8B model
        dict(name="glue_8b", kind="glue", M=8192, D=4096, H=14336),
        # a small block (the head counts of the tests scaled up to a 1B-class width) on three sequences of 336
        # tokens under delayed scaling: token count and hidden width are no powers of two
        dict(name="block_small_delayed", kind="block", B=3, S=336, D=1024, H=2816, Hq=8, Hkv=2, scaling="delayed", e5m2=False),
        # one block of the 8B model on one sequence of 8192 tokens, the paper's training shape
        dict(name="block_8b", kind="block", B=1, S=8192, D=4096, H=14336, Hq=32, Hkv=8, scaling="dynamic", e5m2=False),
    ]


def _log_uniform(rng, lo, hi, step):
    """A multiple of `step` in lo .. hi, spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi, max(lo, int(round(v / step)) * step))


def _width(rng, lo, hi):
    # model widths are mostly multiples of 256, some of 64, a few of 16 only
    return _log_uniform(rng, lo, hi, rng.choice((256, 256, 256, 64, 16)))


def draw(rng):
    kind = rng.choice(("linear", "linear", "linear", "linear", "forward", "attention", "attention", "glue", "block"))
    if kind == "linear":
        while True:
            M, K, N = _log_uniform(rng, 128, 16384, 16), _width(rng, 256, 16384), _width(rng, 256, 16384)
            if M * K * N <= 16384 * 4096 * 14336 / 4:
                break
        scaling = rng.choice(("dynamic", "dynamic", "delayed"))
        rowwise = scaling == "dynamic" and rng.random() < 0.25
        c = _linear("", M, K, N, scaling, rowwise, rng.random() < 0.3)
    elif kind == "forward":
        c = _linear("", _log_uniform(rng, 16, 512, 16), _width(rng, 1024, 8192), _width(rng, 1024, 8192), step=False)
    elif kind == "attention":
        S = _log_uniform(rng, 128, 8192, rng.choice((8, 8, 256)))
        Hkv = rng.choice((2, 4, 8))
        c = dict(kind="attention", B=rng.randint(1, max(1, min(8, 8192 // S))), S=S, Hq=Hkv * rng.choice((1, 2, 4)), Hkv=Hkv)
        if (c["B"] * c["S"]) % 16:
            c["S"] += 8
    elif kind == "glue":
        D = _width(rng, 512, 8192)
        c = dict(kind="glue", M=_log_uniform(rng, 64, 8192, 16), D=D, H=_width(rng, 1024, 14336))
    else:
        heads = rng.choice((4, 8, 16))
        S = _log_uniform(rng, 128, 4096, rng.choice((16, 128)))
        c = dict(kind="block", B=rng.randint(1, max(1, min(4, 4096 // S))), S=S, D=heads * HD, H=_width(rng, 2 * heads * HD, 4 * heads * HD),
                 Hq=heads, Hkv=heads // rng.choice((1, 2, 4)), scaling=rng.choice(("dynamic", "delayed")), e5m2=rng.random() < 0.3)
    c.pop("name", None)
    return c


# ---- inputs -------------------------------------------------------------------------------

def _normal(shape, std, seed, salt):
    g = torch.Generator("cuda")
    g.manual_seed(1000 * seed + salt)
    return (torch.randn(shape, generator=g, dtype=torch.float32, device="cuda") * std).to(torch.bfloat16)


def _linear_inputs(c, seed):
    X = _normal((c["M"], c["K"]), 1.0, seed, 0)
    W = _normal((c["N"], c["K"]), 0.02, seed, 1)
    dY = _normal((c["M"], c["N"]), 1e-3, seed, 2) if c["step"] else None
    return X, W, dY


def _attention_inputs(c, seed):
    M = c["B"] * c["S"]
    return (_normal((M, (c["Hq"] + 2 * c["Hkv"]) * HD), 1.0, seed, 0), _normal((M, c["Hq"] * HD), 1e-3, seed, 1))


def _glue_inputs(c, seed):
    M, D, H = c["M"], c["D"], c["H"]
    return dict(x=_normal((M, D), 1.0, seed, 0), g=(1.0 + _normal((D,), 0.1, seed, 1).float()).to(torch.bfloat16),
                ab=_normal((M, 2 * H), 1.0, seed, 2), dh=_normal((M, H), 1e-3, seed, 3), dy=_normal((M, D), 1e-3, seed, 4),
                res=_normal((M, D), 1e-3, seed, 5))


def _block_inputs(c, seed):
    M, D, H = c["B"] * c["S"], c["D"], c["H"]
    w = dict(g1=torch.ones(D, dtype=torch.bfloat16, device="cuda"), g2=torch.ones(D, dtype=torch.bfloat16, device="cuda"),
             Wqkv=_normal(((c["Hq"] + 2 * c["Hkv"]) * HD, D), 0.05, seed, 2), Wo=_normal((D, D), 0.02, seed, 3),
             W13=_normal((2 * H, D), 0.02, seed, 4), W2=_normal((D, H), 0.02, seed, 5))
    return _normal((M, D), 1.0, seed, 0), w, _normal((M, D), 1e-3, seed, 1)


def _seed_history(hist, scale, amax, fmt):
    """A history as a program in mid-training has it: full, here of this tensor's own amax."""
    for _ in range(hist.numel()):
        f8.amax_history_push(hist, amax, fmt, scale)


def _prepare_linear(c, seed):
    M, K, N = c["M"], c["K"], c["N"]
    gf = f8.E5M2 if c["e5m2"] else f8.E4M3
    X, W, dY = _linear_inputs(c, seed)
    big = max(M, K, N)
    E = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda")
    s = dict(case=c, X=X, W=W, dY=dY, desc=f8.linear_desc(M, K, N, c["rowwise"], gf), saved=f8.Saved(M, K, N, c["rowwise"]),
             ws=f8.new_workspace(big, big), Y=E(M, N))
    if c["step"]:
        s.update(dX=E(M, K), dW=E(N, K))
    else:
        f8.linear_fwd(s["desc"], X, W, s["Y"], s["saved"], s["ws"])  # leaves the weight's codes in saved.w
    if c["scaling"] == "delayed":
        st = s["state"] = f8.ScalingState(f8.DELAYED, HISTORY)
        a = torch.empty(1, dtype=torch.float32, device="cuda")
        for t, h, sc, fmt in ((X, st.hist_x, st.scale_x, f8.E4M3), (W, st.hist_w, st.scale_w, f8.E4M3), (dY, st.hist_dy, st.scale_dy, gf)):
            f8.amax(t, f8.TENSORWISE, a, s["ws"])
            _seed_history(h, sc, a, fmt)
    return s


def _prepare_attention(c, seed):
    B, S, Hq, Hkv = c["B"], c["S"], c["Hq"], c["Hkv"]
    M = B * S
    qkv, do = _attention_inputs(c, seed)
    bf = dict(dtype=torch.bfloat16, device="cuda")
    f32 = dict(dtype=torch.float32, device="cuda")
    E = lambda *s: torch.empty(s, **bf)
    return dict(case=c, qkv=qkv, do=do, qr=E(M, Hq * HD), kr=E(M, Hkv * HD), qt=E(Hq * HD, M), kt=E(Hkv * HD, M), vt=E(Hkv * HD, M),
                o=E(M, Hq * HD), lse=torch.empty((Hq, M), **f32), amax=torch.empty(1, **f32), dot=E(Hq * HD, M), dqr=E(M, Hq * HD),
                dkr=E(M, Hkv * HD), dqkv=E(M, (Hq + 2 * Hkv) * HD), delta=torch.empty((Hq, M), **f32),
                ws=torch.empty(max(16, f8.sdpa_bwd_workspace_bytes(B, S, Hq, Hkv, HD)), dtype=torch.uint8, device="cuda"))


def _prepare_glue(c, seed):
    M, D, H = c["M"], c["D"], c["H"]
    E = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda")
    F = lambda n: torch.empty(n, dtype=torch.float32, device="cuda")
    s = _glue_inputs(c, seed)
    big = max(M, D, 2 * H)
    s.update(case=c, y=E(M, D), rstd=F(M), a_y=F(1), h=E(M, H), a_h=F(1), dab=E(M, 2 * H), a_dab=F(1), dx=E(M, D), dg=F(D), a_dx=F(1),
             ws=f8.new_workspace(big, big))
    return s


def _new_block(c, scaling):
    return TransformerBlock(c["B"], c["S"], c["D"], c["H"], c["Hq"], c["Hkv"], HD, EPS, THETA, f8.E5M2 if c["e5m2"] else f8.E4M3,
                            scaling=scaling, history_len=HISTORY)


def _prepare_block(c, seed):
    x, w, dout = _block_inputs(c, seed)
    blk = _new_block(c, c["scaling"])
    if c["scaling"] == "delayed":
        # the amax of every tensor from one step under dynamic scaling, as a program's first step takes it
        first = _new_block(c, "dynamic")
        first.forward(x, w)
        first.backward(x, w, dout)
        for st, sv in ((blk.st_qkv, first.s_qkv), (blk.st_o, first.s_o), (blk.st_13, first.s_13), (blk.st_2, first.s_2)):
            _seed_history(st.hist_x, st.scale_x, sv.x.amax, f8.E4M3)
            _seed_history(st.hist_w, st.scale_w, sv.w.amax, f8.E4M3)
            _seed_history(st.hist_dy, st.scale_dy, sv.dy.amax, f8.E5M2 if c["e5m2"] else f8.E4M3)
    return dict(case=c, blk=blk, x=x, w=w, dout=dout)


def prepare(case, seed):
    return {"linear": _prepare_linear, "attention": _prepare_attention, "glue": _prepare_glue, "block": _prepare_block}[case["kind"]](case, seed)


# ---- one pass -----------------------------------------------------------------------------

def _run_linear(s):
    c, sv = s["case"], s["saved"]
    if not c["step"]:
        f8.linear_fwd_wq(s["desc"], s["X"], s["Y"], sv, s["ws"])
        return dict(Y=s["Y"], x_codes=sv.x.q, x_scale=sv.x.scale)
    if c["scaling"] == "delayed":
        st = s["state"]
        f8.linear_fwd_scaled(s["desc"], st, s["X"], s["W"], s["Y"], sv, s["ws"])
        f8.linear_bwd_scaled(s["desc"], st, s["dY"], sv, s["dX"], s["dW"], s["ws"])
        return dict(Y=s["Y"], dX=s["dX"], dW=s["dW"], scales=[st.scale_x, st.scale_w, st.scale_dy],
                    hist=[st.hist_x, st.hist_w, st.hist_dy])
    f8.linear_fwd(s["desc"], s["X"], s["W"], s["Y"], sv, s["ws"])
    f8.linear_bwd(s["desc"], s["dY"], sv, s["dX"], s["dW"], s["ws"])
    return dict(Y=s["Y"], dX=s["dX"], dW=s["dW"], codes=[sv.x.q, sv.w.q, sv.dy.q], scales=[sv.x.scale, sv.w.scale, sv.dy.scale])



def _run_attention(s):
    c = s["case"]
    B, S, Hq, Hkv = c["B"], c["S"], c["Hq"], c["Hkv"]
    cut = lambda t: (t[:, :Hq * HD], t[:, Hq * HD:(Hq + Hkv) * HD], t[:, (Hq + Hkv) * HD:])
    q, k, v = cut(s["qkv"])
    dq, dk, dv = cut(s["dqkv"])
    f8.rope(q, S, Hq, HD, s["qr"], s["qt"], THETA)
    f8.rope(k, S, Hkv, HD, s["kr"], s["kt"], THETA)
    f8.transpose_bf16(v, s["vt"])
    f8.sdpa_fwd(s["qr"], s["kr"], s["vt"], B, S, Hq, Hkv, HD, s["o"], s["lse"], None, s["amax"])
    f8.transpose_bf16(s["do"], s["dot"])
    f8.sdpa_bwd(s["qr"], s["qt"], s["kr"], s["kt"], v, s["o"], s["do"], s["dot"], s["lse"], B, S, Hq, Hkv, HD, s["dqr"], s["dkr"], dv,
                s["delta"], s["ws"])
    f8.rope(s["dqr"], S, Hq, HD, dq, None, THETA, True)
    f8.rope(s["dkr"], S, Hkv, HD, dk, None, THETA, True)
    return dict(o=s["o"], lse=s["lse"], amax=s["amax"], dqkv=s["dqkv"])


def _run_glue(s):
    f8.rmsnorm(s["x"], s["g"], EPS, s["y"], s["rstd"], s["a_y"], s["ws"])
    f8.silu_mul(s["ab"], s["h"], s["a_h"], s["ws"])
    f8.silu_mul_bwd(s["ab"], s["dh"], s["dab"], s["a_dab"], s["ws"])
    s["a_dx"].zero_()  # the call raises it to the amax of what it writes
    f8.rmsnorm_bwd_add(s["x"], s["g"], s["rstd"], s["dy"], s["res"], s["dx"], s["dg"], s["ws"], None, s["a_dx"])
    return dict(y=s["y"], rstd=s["rstd"], h=s["h"], dab=s["dab"], dx=s["dx"], dg=s["dg"], amax=[s["a_y"], s["a_h"], s["a_dab"], s["a_dx"]])


def _run_block(s):
    b = s["blk"]
    out = b.forward(s["x"], s["w"])
    dx = b.backward(s["x"], s["w"], s["dout"])
    return dict(out=out, dx=dx, dWqkv=b.dWqkv, dWo=b.dWo, dW13=b.dW13, dW2=b.dW2, dg1=b.dg1, dg2=b.dg2)


def run(state):
    return {"linear": _run_linear, "attention": _run_attention, "glue": _run_glue, "block": _run_block}[state["case"]["kind"]](state)


# ---- what a pass cannot do without ----------------------------------------------------------

def _attention_flops(B, S, Hq):
    fwd = 4 * B * S * S * Hq * HD // 2  # causal half of the two products
    return fwd + 5 * fwd // 2           # and the five products of the backward


def work(case):
    c = case
    if c["kind"] == "linear":
        M, K, N = c["M"], c["K"], c["N"]
        if not c["step"]:  # X in, Y out in bf16, the kept weight codes in
            return {"bytes": 2 * M * K + 2 * M * N + N * K, "flops": 2 * M * K * N}
        return {"bytes": 2 * (2 * M * K + 2 * M * N + 2 * N * K), "flops": 6 * M * K * N}
    if c["kind"] == "attention":
        B, S, Hq, Hkv = c["B"], c["S"], c["Hq"], c["Hkv"]
        M = B * S
        return {"bytes": 2 * M * HD * (2 * (Hq + 2 * Hkv) + 2 * Hq) + 4 * M * Hq, "flops": _attention_flops(B, S, Hq)}
    if c["kind"] == "glue":
        M, D, H = c["M"], c["D"], c["H"]
        # x, dy, res in, y, dx out; a, b, dh in, h, da, db out
        return {"bytes": 2 * M * 5 * D + 2 * M * 6 * H, "flops": 0}
    B, S, D, H, Hq, Hkv = (c[k] for k in ("B", "S", "D", "H", "Hq", "Hkv"))
    M, weights = B * S, (Hq + 2 * Hkv) * HD * D + D * D + 3 * D * H
    return {"bytes": 2 * 2 * weights + 2 * 4 * M * D, "flops": 6 * M * weights + _attention_flops(B, S, Hq)}


def tolerance(case):
    # Measured against exact(): 1.7e-3 for what is rounded to bf16 once (linear, glue), 2.8e-3 for the attention; a
    # chain of fp8 linears is 1 to 5e-2 off, since a value that rounds the other way moves codes further down.
    return {"linear": {"rel": 7e-3}, "attention": {"rel": 1.5e-2}, "glue": {"rel": 7e-3}, "block": {"rel": 3e-2}}[case["kind"]]


# ---- the same in 64 bits ----------------------------------------------------------------------
# The fp8 codes and the bf16 tensors that calls hand to each other are part of what an entry point defines, so
# they are formed here too; everything between them is in 64 bits.

def _bf(t):
    return t.to(torch.bfloat16).double()


def _quantised(t, fmt, dim=None):
    """The values that the fp8 codes of t stand for: code / scale with scale = FMAX / amax in fp32."""
    t = t.float()
    a = t.abs().amax() if dim is None else t.abs().amax(dim, keepdim=True)
    a = torch.clamp(a, min=1e-12)
    s = torch.full_like(a, FMAX[fmt]) / a  # one rounded division (number / tensor would multiply by a reciprocal)
    return torch.clamp(t * s, -FMAX[fmt], FMAX[fmt]).to(F8_TYPE[fmt]).double() * (1.0 / s).double()


def _exact_linear(c, seed):
    X, W, dY = _linear_inputs(c, seed)
    gf = f8.E5M2 if c["e5m2"] else f8.E4M3
    rows, cols = (1, 0) if c["rowwise"] else (None, None)
    Y = _quantised(X, f8.E4M3, rows) @ _quantised(W, f8.E4M3, rows).t()
    if not c["step"]:
        return dict(Y=Y, x_codes=None, x_scale=None)
    dX = _quantised(dY, gf, rows) @ _quantised(W, f8.E4M3, cols)
    dW = _quantised(dY, gf, cols).t() @ _quantised(X, f8.E4M3, cols)
    return dict(Y=Y, dX=dX, dW=dW)


def _rotate(t, S, inverse):
    M, w = t.shape
    x = t.double().view(M, w // HD, HD // 2, 2)
    f = THETA ** (-2.0 * torch.arange(HD // 2, dtype=torch.float64, device=t.device) / HD)
    a = (torch.arange(M, device=t.device) % S).double()[:, None] * f[None, :] * (-1.0 if inverse else 1.0)
    c, s = torch.cos(a)[:, None, :], torch.sin(a)[:, None, :]
    return torch.stack((x[..., 0] * c - x[..., 1] * s, x[..., 0] * s + x[..., 1] * c), dim=-1).view(M, w)


def _head(t, b, S, h):
    return t[b * S:(b + 1) * S, h * HD:(h + 1) * HD]


def _scores(q, k, b, S, h, kv):
    s = _head(q, b, S, h) @ _head(k, b, S, kv).t() / math.sqrt(HD)
    return s.masked_fill_(torch.ones((S, S), dtype=torch.bool, device=s.device).triu_(1), -math.inf)


def _attention_fwd(q, k, v, B, S, Hq, Hkv):
    o, lse = torch.empty_like(q), torch.empty((Hq, q.shape[0]), dtype=torch.float64, device=q.device)
    for b in range(B):
        for h in range(Hq):
            s = _scores(q, k, b, S, h, h // (Hq // Hkv))
            l = torch.logsumexp(s, 1)
            lse[h, b * S:(b + 1) * S] = l
            _head(o, b, S, h).copy_(s.sub_(l[:, None]).exp_() @ _head(v, b, S, h // (Hq // Hkv)))
    return o, lse


def _attention_bwd(q, k, v, o, do, lse, B, S, Hq, Hkv):
    dq, dk, dv = torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v)
    for b in range(B):
        for h in range(Hq):
            kv = h // (Hq // Hkv)
            d = _head(do, b, S, h)
            p = _scores(q, k, b, S, h, kv).sub_(lse[h, b * S:(b + 1) * S, None]).exp_()
            _head(dv, b, S, kv).add_(p.t() @ d)
            ds = p.mul_((d @ _head(v, b, S, kv).t()).sub_((d * _head(o, b, S, h)).sum(1, keepdim=True)))
            _head(dq, b, S, h).copy_(ds @ _head(k, b, S, kv) / math.sqrt(HD))
            _head(dk, b, S, kv).add_(ds.t() @ _head(q, b, S, h) / math.sqrt(HD))
    return dq, dk, dv


def _middle_fwd(qkv, B, S, Hq, Hkv):
    a, b = Hq * HD, (Hq + Hkv) * HD
    q, k, v = _bf(_rotate(qkv[:, :a], S, False)), _bf(_rotate(qkv[:, a:b], S, False)), qkv[:, b:].double()
    o, lse = _attention_fwd(q, k, v, B, S, Hq, Hkv)
    return q, k, v, o, lse


def _middle_bwd(q, k, v, o, do, lse, B, S, Hq, Hkv):
    dq, dk, dv = _attention_bwd(q, k, v, _bf(o), do, lse, B, S, Hq, Hkv)
    return torch.cat((_rotate(_bf(dq), S, True), _rotate(_bf(dk), S, True), dv), dim=1)


def _exact_attention(c, seed):
    a = (c["B"], c["S"], c["Hq"], c["Hkv"])
    qkv, do = _attention_inputs(c, seed)
    q, k, v, o, lse = _middle_fwd(qkv, *a)
    return dict(o=o, lse=lse, amax=None, dqkv=_middle_bwd(q, k, v, o, do.double(), lse, *a))


def _norm_fwd(x, g):
    r = 1.0 / torch.sqrt(x.square().mean(1, keepdim=True) + EPS)
    return x * r * g, r


def _norm_bwd(x, g, r, dy):
    gd = g * dy
    return r * gd - x * r ** 3 * (x * gd).mean(1, keepdim=True), (dy * x * r).sum(0)


def _gate_bwd(a, b, dh):
    s = torch.sigmoid(a)
    return torch.cat((dh * b * s * (1.0 + a * (1.0 - s)), dh * a * s), dim=1)


def _exact_glue(c, seed):
    t = {k: v.double() for k, v in _glue_inputs(c, seed).items()}
    y, r = _norm_fwd(t["x"], t["g"])
    a, b = t["ab"][:, :c["H"]], t["ab"][:, c["H"]:]
    dx, dg = _norm_bwd(t["x"], t["g"], r, t["dy"])
    return dict(y=y, rstd=r[:, 0], h=a * torch.sigmoid(a) * b, dab=_gate_bwd(a, b, t["dh"]), dx=t["res"] + _bf(dx), dg=dg, amax=None)


def _exact_block(c, seed):
    a4 = (c["B"], c["S"], c["Hq"], c["Hkv"])
    gf, H = f8.E5M2 if c["e5m2"] else f8.E4M3, c["H"]
    x, w, dout = _block_inputs(c, seed)
    x, dout, g1, g2 = x.double(), dout.double(), w["g1"].double(), w["g2"].double()
    W = {n: _quantised(w[n], f8.E4M3) for n in ("Wqkv", "Wo", "W13", "W2")}
    xn, r1 = _norm_fwd(x, g1)
    xn8 = _quantised(_bf(xn), f8.E4M3)
    qkv = _bf(xn8 @ W["Wqkv"].t())
    q, k, v, o, lse = _middle_fwd(qkv, *a4)
    o8 = _quantised(_bf(o), f8.E4M3)
    h1 = _bf(x + _bf(o8 @ W["Wo"].t()))
    hn, r2 = _norm_fwd(h1, g2)
    hn8 = _quantised(_bf(hn), f8.E4M3)
    ab = _bf(hn8 @ W["W13"].t())
    a, b = ab[:, :H], ab[:, H:]
    hh8 = _quantised(_bf(a * torch.sigmoid(a) * b), f8.E4M3)
    out = h1 + _bf(hh8 @ W["W2"].t())
    d8 = _quantised(dout, gf)
    dhh, dW2 = _bf(d8 @ W["W2"]), d8.t() @ hh8
    d8 = _quantised(_bf(_gate_bwd(a, b, dhh)), gf)
    dhn, dW13 = _bf(d8 @ W["W13"]), d8.t() @ hn8
    dh1, dg2 = _norm_bwd(h1, g2, r2, dhn)
    dh1 = _bf(dout + _bf(dh1))
    d8 = _quantised(dh1, gf)
    datt, dWo = _bf(d8 @ W["Wo"]), d8.t() @ o8
    d8 = _quantised(_bf(_middle_bwd(q, k, v, o, datt, lse, *a4)), gf)
    dxn, dWqkv = _bf(d8 @ W["Wqkv"]), d8.t() @ xn8
    dx, dg1 = _norm_bwd(x, g1, r1, dxn)
    return dict(out=out, dx=dh1 + _bf(dx), dWqkv=dWqkv, dWo=dWo, dW13=dW13, dW2=dW2, dg1=dg1, dg2=dg2)


def exact(case, seed):
    return {"linear": _exact_linear, "attention": _exact_attention, "glue": _exact_glue, "block": _exact_block}[case["kind"]](case, seed)
