"""The work a user has the library do, as measurable cases.

A case is one call pattern of the public binding (paper_2608_21308_amd.e2ttt):

  apply    streaming decode: the net of every unit at its chunk-start state for
           the arriving token(s) (e2ttt.apply into the loop's own buffers)
  forward  prefill, and the state update of decode once a chunk has filled
           (e2ttt.forward into the program's own buffers and workspace)
  train    a training step of the layer: gates from their logits, the chunk
           chain, and the backward of both (GatesFunction and E2TTTFunction
           under torch.autograd; with the LayerNorm affine, which the autograd
           wrapper does not take, the binding's forward and backward)

Inputs: queries and keys of unit length (the paper normalises both), values
that a head can learn (a per-head linear map of the key plus noise, about unit
variance per element as a projection gives), gates from N(0, 1) logits through
the paper's own parameterization (eta_base 0.01, tau 32, alpha_base 0.1), and
initial fast weights at the usual 1/sqrt(fan-in) scale.  With these the chunk
chain carries a rounding error along instead of multiplying it, so outputs can
be compared over hundreds of chunks.
"""
import math

import torch

from paper_2608_21308_amd import e2ttt

FLAG_AFFINE = e2ttt.FLAG_LN_AFFINE
FLAG_POST_NORM = e2ttt.FLAG_POST_NORM


def _case(name, kind, fw, B, H, T, d, dh, C, io="bf16", affine=False, post_norm=False,
          decay=True):
    c = dict(kind=kind, fw=fw, B=B, H=H, T=T, d=d, dh=dh, C=C, io=io, affine=affine,
             post_norm=post_norm, decay=decay)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # decode of eight sequences, one token each: the call made for every token
        _case("decode_mlp_b8", "apply", "mlp", 8, 16, 1, 64, 256, 64),
        # decode of one sequence at the 1.3B model's head dim, SwiGLU at its 8/3 width
        _case("decode_swiglu_d128_b1", "apply", "swiglu", 1, 16, 1, 128, 344, 512),
        # the state update of that decode when 64 tokens have arrived (one chunk)
        _case("advance_mlp_b8", "forward", "mlp", 8, 16, 64, 64, 256, 64),
        # prefill of two 2k prompts on four heads (a tensor-parallel slice)
        _case("prefill_mlp_b2h4", "forward", "mlp", 2, 4, 2048, 64, 256, 64),
        # long-context prefill: 512 chunks in sequence on the layer's sixteen heads
        _case("prefill_mlp_32k", "forward", "mlp", 1, 16, 32768, 64, 256, 64),
        # the same with the SwiGLU net at 8k (over many more chunks than these its residual
        # LayerNorm form multiplies rounding, so that nothing could be compared)
        _case("prefill_swiglu_8k", "forward", "swiglu", 1, 16, 8192, 64, 172, 64),
        # a training step of a slice of heads, SwiGLU net
        _case("train_swiglu_b2h4", "train", "swiglu", 2, 4, 2048, 64, 172, 64),
        # a training step of the 1.3B layer shape, sixteen heads of 64, batch 8
        _case("train_mlp_1p3b", "train", "mlp", 8, 16, 4096, 64, 256, 64),
        # the paper's throughput shape: heads of 128, chunks of 512, batch 2
        _case("train_mlp_d128_c512", "train", "mlp", 2, 16, 2048, 128, 512, 512),
        # the same layer with the SwiGLU net on one ragged sequence
        _case("train_swiglu_d128_ragged", "train", "swiglu", 1, 16, 1500, 128, 344, 512),
        # the paper's training options (affine, post-chunk normalisation), odd batch,
        # ragged chunks longer than the tile, a width that is no multiple of the tile
        _case("train_mlp_options", "train", "mlp", 3, 5, 1000, 64, 120, 100, affine=True,
              post_norm=True),
        # float32 debugging and small-head configuration
        _case("train_mlp_f32", "train", "mlp", 2, 4, 515, 16, 64, 16, io="f32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above."""
    kind = rng.choice(["apply", "forward", "forward", "train", "train", "train"])
    fw = rng.choice(["mlp", "mlp", "swiglu"])
    io, d = rng.choice([("bf16", 64)] * 4 + [("bf16", 128)] * 2 + [("f32", 16)])
    widest = {64: 256 if fw == "mlp" else 192, 128: 512, 16: 128}[d]
    dh = _log_int(rng, d, widest)
    B, H = _log_int(rng, 1, 8), rng.choice([1, 4, 5, 8, 12, 16])
    C = rng.choice([16, 48, 64, 64, 100, 128, 256, 512])
    if kind == "apply":
        return _case(None, kind, fw, B, H, rng.choice([1, 1, 1, 2, 5, 16]), d, dh, C, io)
    # (SwiGLU multiplies rounding by chunk and under the normalisation, see listed())
    most = min(4096 if fw == "mlp" else 32 * max(C, 64), 4096, 262144 // (B * H))
    T = C if kind == "forward" and rng.random() < 0.3 else _log_int(rng, 200, most)
    opts = kind == "train" and rng.random() < 0.25
    return _case(None, kind, fw, B, H, T, d, dh, C, io, affine=opts and rng.random() < 0.6,
                 post_norm=opts and fw == "mlp" and rng.random() < 0.6, decay=rng.random() < 0.85)


# ------------------------------------------------------------------- inputs
def _cfg(c):
    flags = (FLAG_AFFINE if c["affine"] else 0) | (FLAG_POST_NORM if c["post_norm"] else 0)
    return e2ttt.Config(c["B"], c["H"], c["T"], c["d"], c["dh"], c["C"],
                        e2ttt.FW_MLP if c["fw"] == "mlp" else e2ttt.FW_SWIGLU,
                        e2ttt.DT_BF16 if c["io"] == "bf16" else e2ttt.DT_F32, flags)


def _inputs(c, seed):
    """Everything the case reads, as float32 / io-type tensors, from the seed alone."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(int(seed))
    B, H, T, d, dh = c["B"], c["H"], c["T"], c["d"], c["dh"]
    io = torch.bfloat16 if c["io"] == "bf16" else torch.float32

    def randn(*s):
        return torch.randn(*s, device=dev, generator=g)

    def unit():
        x = randn(B, H, T, d)
        return (x / x.norm(dim=-1, keepdim=True)).to(io)

    n1 = (1 if c["fw"] == "mlp" else 2) * dh * d
    w = torch.cat([randn(H, n1) / math.sqrt(d), randn(H, d * dh) / math.sqrt(dh)], 1)
    x = dict(q=unit(), w_in=w.expand(B, H, -1).contiguous())
    if c["affine"]:
        x["ln_weight"], x["ln_bias"] = 1.0 + 0.1 * randn(H, d), 0.1 * randn(H, d)
    if c["kind"] == "apply":
        return x
    x["k"] = unit()
    recall = torch.matmul(x["k"].float(), randn(H, d, d))
    x["v"] = (0.8 * recall + 0.6 * randn(B, H, T, d)).to(io)
    for n in ("l_eta", "l_beta", "l_alpha") if c["decay"] else ("l_eta", "l_beta"):
        x[n] = randn(B, H, T)
    if c["kind"] == "train":
        x["d_out"] = randn(B, H, T, d).to(io)
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    s = dict(case=case, cfg=_cfg(case), gate=e2ttt.GateParams(), **x)
    if case["kind"] == "apply":
        s["out"] = torch.empty_like(x["q"])
    elif case["kind"] == "forward":
        # the gates of a prompt, and the buffers a serving loop keeps
        s["eta"], s["beta"], s["gamma"] = e2ttt.gates_forward(s["gate"], x["l_eta"], x["l_beta"],
                                                              x.get("l_alpha"))
        s["buf"] = dict(out=torch.empty_like(x["q"]), w_out=torch.empty_like(x["w_in"]),
                        m_out=torch.empty_like(x["w_in"]),
                        workspace=e2ttt.alloc_workspace(s["cfg"], False))
    else:
        for n in ("q", "k", "v", "l_eta", "l_beta", "l_alpha", "w_in"):
            if n in s:
                s[n].requires_grad_(not case["affine"])
    return s


def run(s):
    kind, cfg = s["case"]["kind"], s["cfg"]
    if kind == "apply":
        return e2ttt.apply(cfg, s["q"], s["w_in"], out=s["out"], ln_weight=s.get("ln_weight"),
                           ln_bias=s.get("ln_bias"))
    if kind == "forward":
        out, w_out, m_out, _ = e2ttt.forward(cfg, s["q"], s["k"], s["v"], s["eta"], s["beta"],
                                             s["gamma"], s["w_in"], None, **s["buf"])
        return dict(out=out, w_out=w_out, m_out=m_out)
    if s["case"]["affine"]:
        return _train_affine(s)
    names = [n for n in ("q", "k", "v", "l_eta", "l_beta", "l_alpha", "w_in") if n in s]
    eta, beta, gamma = e2ttt.GatesFunction.apply(s["gate"], s["l_eta"], s["l_beta"],
                                                 s.get("l_alpha"))
    out, w_out, m_out = e2ttt.E2TTTFunction.apply(cfg, s["q"], s["k"], s["v"], eta, beta, gamma,
                                                  s["w_in"], None)
    grads = torch.autograd.grad([out], [s[n] for n in names], [s["d_out"]])
    return dict(out=out.detach(), w_out=w_out.detach(), m_out=m_out.detach(),
                **{"d_" + n: g for n, g in zip(names, grads)})


def _train_affine(s):
    cfg, ln = s["cfg"], dict(ln_weight=s["ln_weight"], ln_bias=s["ln_bias"])
    logits = s["l_eta"], s["l_beta"], s.get("l_alpha")
    eta, beta, gamma = e2ttt.gates_forward(s["gate"], *logits)
    args = s["q"], s["k"], s["v"], eta, beta, gamma, s["w_in"], None
    out, w_out, m_out, ws = e2ttt.forward(cfg, *args, save_for_backward=True, **ln)
    g = e2ttt.backward(cfg, *args, ws, s["d_out"], **ln)
    dl = e2ttt.gates_backward(s["gate"], *logits, g["d_eta"], g["d_beta"], g["d_gamma"])
    res = dict(out=out, w_out=w_out, m_out=m_out, d_q=g["dq"], d_k=g["dk"], d_v=g["dv"],
               d_l_eta=dl[0], d_l_beta=dl[1], d_w_in=g["d_w_in"], d_ln_weight=g["d_ln_weight"],
               d_ln_bias=g["d_ln_bias"])
    if dl[2] is not None:
        res["d_l_alpha"] = dl[2]
    return res


# ------------------------------------------------------------ what it costs
def work(c):
    """Inputs read once and outputs written once; contractions of 2 d dh per token.

    Forward, per token: the net on the key and on the query, its gradient's one
    contraction through the second layer, and two aggregations per matrix.  The
    backward of contractions takes twice their operations."""
    U, T, d, dh = c["B"] * c["H"], c["T"], c["d"], c["dh"]
    nmat = 2 if c["fw"] == "mlp" else 3
    e = 2 if c["io"] == "bf16" else 4
    tok, row, state = U * T, U * T * d * e, U * nmat * d * dh * 4
    unit = 2.0 * d * dh * tok
    if c["kind"] == "apply":
        return {"bytes": 2 * row + state, "flops": nmat * unit}
    gates = 3 if c["decay"] else 2
    fwd = 2 * nmat + 1 + 2 * nmat
    if c["kind"] == "forward":
        return {"bytes": 4 * row + gates * 4 * tok + 3 * state, "flops": fwd * unit}
    return {"bytes": (4 + 4) * row + 2 * gates * 4 * tok + (3 + 1) * state, "flops": 3 * fwd * unit}


def tolerance(c):
    """About four times the largest error against exact() over listed and drawn cases: apply
    1.7e-3 (the bf16 rounding of the output) and below 1e-6; the float32 chain 4e-6; the bf16
    chain 1e-2 at the end of its longest chains (1.8e-2 at gradients whose terms cancel)."""
    if c["kind"] == "apply":
        return {"rel": 7e-3} if c["io"] == "bf16" else {"rel": 4e-6}
    return {"rel": 2e-5} if c["io"] == "f32" else {"rel": 3e-2}


# ------------------------------------------------------------ in 64 bits
def _t(x):
    return x.transpose(-1, -2)


def _matrices(w, c):
    d, dh = c["d"], c["dh"]
    n1 = 1 if c["fw"] == "mlp" else 2
    m = [w[:, i * dh * d:(i + 1) * dh * d].reshape(-1, dh, d) for i in range(n1)]
    return m + [w[:, n1 * dh * d:].reshape(-1, d, dh)]


def _net(ms, x, c):
    """Hidden activations, their derivatives' factors, and y of the bare net."""
    h = [x @ _t(m) for m in ms[:-1]]
    if c["fw"] == "mlp":
        cdf = 0.5 * (1.0 + torch.erf(h[0] / math.sqrt(2.0)))
        a = h[0] * cdf
        d1 = [cdf + h[0] * torch.exp(-0.5 * h[0] * h[0]) / math.sqrt(2.0 * math.pi)]
    else:
        s = torch.sigmoid(h[0])
        a = h[0] * s * h[1]
        d1 = [h[1] * s * (1.0 + h[0] * (1.0 - s)), h[0] * s]
    return a, d1, a @ _t(ms[-1])


def _ln(y):
    y = y - y.mean(-1, keepdim=True)
    r = (y.square().mean(-1, keepdim=True) + 1e-5).rsqrt()
    return y * r, r


def _chunk(c, nmat, q, k, v, kw, km, cw, cm, cb, la, lb, *state):
    """One chunk at its start state: outputs and the state after it (Algorithm 1)."""
    ms, mm, w0 = state[:nmat], state[nmat:2 * nmat], state[2 * nmat:]
    a, d1, y = _net(ms, k, c)
    z, r = _ln(y)
    e = (v - k - la * z - lb) * la
    dy = (e - e.mean(-1, keepdim=True) - z * (e * z).mean(-1, keepdim=True)) * r
    dh = [(dy @ ms[-1]) * x for x in d1]
    out = q + la * _ln(_net(ms, q, c)[2])[0] + lb

    def grads(s):
        return [_t(x * s) @ k for x in dh] + [_t(dy * s) @ a]

    ws = [cw * x + cm * m + g for x, m, g in zip(ms, mm, grads(kw[..., None]))]
    ms2 = [cb * m + g for m, g in zip(mm, grads(km[..., None]))]
    if c["post_norm"]:
        ws = [x * (t.norm(dim=-1, keepdim=True) / x.norm(dim=-1, keepdim=True))
              for x, t in zip(ws, w0)]
    return (out, *ws, *ms2)


def _scalars(eta, beta, gamma):
    """The scalar kernels of whole chunks [..., L] (Prop. 1)."""
    def after(x):     # products of the later tokens' factors
        p = x[..., 1:].flip(-1).cumprod(-1).flip(-1)
        return torch.cat([p, torch.ones_like(x[..., :1])], -1)

    bt, gt = after(beta), after(gamma)
    s = [gt[..., -1]]
    for t in range(eta.shape[-1] - 2, -1, -1):
        s.append(gt[..., t] + beta[..., t + 1] * s[-1])
    s = torch.stack(s[::-1], -1)
    return (eta * s, eta * bt, gt[..., 0] * gamma[..., 0], beta[..., 0] * s[..., 0],
            beta[..., 0] * bt[..., 0])


def exact(c, seed):
    from torch.utils.checkpoint import checkpoint
    x = {n: t.double() for n, t in _inputs(c, seed).items()}
    B, H, T, d, C = c["B"], c["H"], c["T"], c["d"], c["C"]
    U, nmat = B * H, 2 if c["fw"] == "mlp" else 3
    train = c["kind"] == "train"
    names = [n for n in ("q", "k", "v", "l_eta", "l_beta", "l_alpha", "w_in", "ln_weight",
                         "ln_bias") if n in x]
    if train:
        for n in names:
            x[n].requires_grad_(True)
    f = {n: t.reshape(U, *t.shape[2:]) for n, t in x.items() if not n.startswith("ln_")}
    if c["affine"]:
        la, lb = (x[n].repeat(B, 1)[:, None, :] for n in ("ln_weight", "ln_bias"))
    else:
        la, lb = torch.ones((), dtype=torch.float64, device="cuda"), 0.0
    w0 = _matrices(f["w_in"], c)
    if c["kind"] == "apply":
        z = _ln(_net(w0, f["q"], c)[2])[0]
        return (f["q"] + la * z + lb).reshape(B, H, T, d)
    eta = 0.01 * torch.sigmoid(f["l_eta"])
    beta = torch.sigmoid(f["l_beta"]) ** (1.0 / 32.0)
    gamma = torch.ones_like(eta)
    if c["decay"]:
        gamma = 1.0 - eta * 0.1 * torch.sigmoid(f["l_alpha"])
    if not train:     # the gates as the call receives them
        eta, beta, gamma = eta.float().double(), beta.float().double(), gamma.float().double()
    full = T // C * C
    parts = []
    if full:
        whole = _scalars(*(t[:, :full].reshape(U, -1, C) for t in (eta, beta, gamma)))
        parts += [[t[:, r] for t in whole] for r in range(full // C)]
    if full < T:
        parts.append(list(_scalars(*(t[:, full:] for t in (eta, beta, gamma)))))
    state = [*w0, *(torch.zeros_like(m) for m in w0)]
    outs = []
    for r, (kw, km, cw, cm, cb) in enumerate(parts):
        sl = slice(r * C, min(T, (r + 1) * C))
        carry = [t[:, None, None] for t in (cw, cm, cb)]
        args = (c, nmat, f["q"][:, sl], f["k"][:, sl], f["v"][:, sl], kw, km, *carry, la, lb,
                *state, *w0)
        res = checkpoint(_chunk, *args, use_reentrant=False) if train else _chunk(*args)
        outs.append(res[0])
        state = list(res[1:])
    out = torch.cat(outs, 1).reshape(B, H, T, d)

    def flat(ms):
        return torch.cat([m.reshape(U, -1) for m in ms], 1).reshape(B, H, -1)

    res = dict(out=out, w_out=flat(state[:nmat]), m_out=flat(state[nmat:]))
    if train:
        g = torch.autograd.grad([out], [x[n] for n in names], [x["d_out"]], allow_unused=True)
        res.update({"d_" + n: torch.zeros_like(x[n]) if t is None else t
                    for n, t in zip(names, g)})
    return {n: t.detach() for n, t in res.items()}
