"""Chains that leave the query side to kernels of their own (head dim 64, bf16,
eight chunks or more of few units) at the sizes where that can go wrong: last
chunks of one token and of a few, chunks shorter and longer than a 32-token
tile, hidden widths that are no multiple of 32, one to three workgroups per
unit, the post-chunk normalisation (also over chunks above 64 tokens) and the
LayerNorm affine; and more chunks than one launch takes without saving (the
state passes through w_out and m_out between launches).  Each case runs the
forward without saving, the forward with saving and the backward against the
fp64 oracle; the bar is that of the other
bf16 tests (2e-2, with the local maxima).  The affine cases draw a tenth of the
usual learning rates: with these a relative change of 2^-9 of the inputs moves
the oracle's results by half the bar at most, with the usual ones by up to
their whole size."""
import numpy as np
import pytest
import torch

from paper_2608_21308_amd import e2ttt, workloads as WL
from tests import fp32ref
from tests.gpu_util import TOL, config_of, to_dev
from tests.test_gpu_ln_affine import affine
from tests.test_gpu_post_norm import errors, run_gpu, run_oracle, with_state

pytestmark = pytest.mark.gpu

BARE, AFF, PN = e2ttt.FLAG_NO_RESIDUAL_LN, e2ttt.FLAG_LN_AFFINE, e2ttt.FLAG_POST_NORM


@pytest.mark.parametrize("fw,dh,B,H,T,C,flags", [
    (0, 64, 1, 2, 113, 16, 0),          # eight chunks, the last of one token
    (0, 100, 3, 3, 236, 33, 0),         # nine units, a second tile of one token
    (0, 128, 1, 1, 510, 64, BARE),      # whole tiles, the last chunk two tokens short
    (0, 250, 1, 3, 127, 5, 0),          # two workgroups, 26 chunks
    (0, 256, 2, 16, 90, 10, PN | BARE), # the most units
    (1, 64, 1, 2, 129, 16, AFF),
    (1, 100, 1, 3, 236, 33, BARE),
    (1, 172, 1, 2, 121, 4, BARE),       # three workgroups, 31 chunks
    (1, 172, 1, 9, 110, 12, PN | AFF),
    (1, 128, 1, 2, 142, 5, PN | AFF),   # 29 chunks, normalised
    (1, 64, 1, 2, 570, 70, PN | AFF),   # chunks of two chain tiles
])
def test_query_side_apart(fw, dh, B, H, T, C, flags):
    w = WL.WORKLOADS[1].with_(fw=fw, B=B, H=H, T=T, d=64, dh=dh, C=C, backward=True,
                              seed=4300 + T + dh)
    x = with_state(WL.make_inputs(w), 7, 1e-2)
    if flags & AFF:
        x["eta"] = x["eta"] * np.float32(0.1)
    ln = affine(H, 64, 11) if flags & AFF else None
    ref = run_oracle(w, x, flags, ln)
    free = run_gpu(w, x, flags, ln, backward=False)
    errs = errors(run_gpu(w, x, flags, ln), ref, x, C)
    errs.update({"%s (not saving)" % n: e for n, e in
                 errors(free, {n: ref[n] for n in free}, x, C).items()})
    print("apart fw=%d dh=%d U=%d T=%d C=%d" % (fw, dh, B * H, T, C),
          {k: "%.2e" % v for k, v in errs.items()}, flush=True)
    bar = {}
    if flags & PN:
        # with the normalisation the adjoint of W is nearly orthogonal to W_0's rows,
        # and d_gamma what little is left of <Wb_C, W_0>: the bar from the case itself
        units = sorted({0, B * H // 2, B * H - 1})
        pick = lambda a: a if a is None else np.ascontiguousarray(
            a.reshape((B * H,) + a.shape[2:])[units][None])
        xs = {n: pick(a) for n, a in x.items()}
        lns = None if ln is None else tuple(np.ascontiguousarray(a[[u % H for u in units]])
                                            for a in ln)
        bar = fp32ref.bf16_state_bar(errors, xs, {n: pick(ref[n]) for n in ("d_beta", "d_gamma")},
                                     C=C, fw=fw, dh=dh, flags=flags, ln=lns)
        print("bars", {n: "%.1e" % b for n, b in bar.items()}, flush=True)
    assert all(e <= bar.get(n, TOL["bf16"]) for n, e in errs.items()), errs


def test_state_in_place():
    # w_out over w_in
    w = WL.WORKLOADS[1].with_(fw=0, B=1, H=2, T=300, d=64, dh=256, C=10, seed=4400)
    cfg = config_of(w)
    t = to_dev(with_state(WL.make_inputs(w), 3, 1e-2), w.io)
    args = t["q"], t["k"], t["v"], t["eta"], t["beta"], t["gamma"]
    ref = e2ttt.forward(cfg, *args, t["w_in"], t["m_in"])[:3]
    ws, ms, out = t["w_in"].clone(), t["m_in"].clone(), torch.empty_like(ref[0])
    e2ttt.forward_static(cfg, *args, ws, ms, out, ws, ms)
    for n, a, b in zip(("out", "w_out", "m_out"), (out, ws, ms), ref):
        assert torch.equal(a, b), n


def test_under_capture():
    # the launches and the query kernel as one graph: every replay equals the
    # eager call
    w = WL.WORKLOADS[1].with_(fw=1, B=1, H=2, T=300, d=64, dh=172, C=10, seed=4500)
    cfg = config_of(w, flags=BARE)
    t = to_dev(with_state(WL.make_inputs(w), 3, 1e-2), w.io)
    args = t["q"], t["k"], t["v"], t["eta"], t["beta"], t["gamma"], t["w_in"], t["m_in"]
    ref = e2ttt.forward(cfg, *args)[:3]
    got = tuple(torch.empty_like(r) for r in ref)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        e2ttt.forward_static(cfg, *args, *got)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        e2ttt.forward_static(cfg, *args, *got)
    for _ in range(4):
        for g in got:
            g.fill_(float("nan"))
        graph.replay()
        eager = e2ttt.forward(cfg, *args)[:3]
        torch.cuda.synchronize()
        for n, a, b, c in zip(("out", "w_out", "m_out"), got, eager, ref):
            assert torch.equal(a, b) and torch.equal(b, c), n


# more chunks than 256 MB of copies hold (85 of 32 units MLP 256, 68 SwiGLU 172,
# 85 of 64 units MLP 128): two and three launches
@pytest.mark.parametrize("fw,dh,U,NC,C,flags", [
    (0, 256, 32, 87, 2, 0),
    (1, 172, 32, 140, 3, BARE),
    (0, 128, 64, 171, 1, PN | BARE),
])
def test_several_launches_equal_one(fw, dh, U, NC, C, flags):
    # saving runs all chunks in one launch; without saving, with the state in
    # place, and as a graph (the launches and the clearing of their flags
    # between): the same numbers
    T = NC * C - (C > 1)
    w = WL.WORKLOADS[1].with_(fw=fw, B=2, H=U // 2, T=T, d=64, dh=dh, C=C, seed=4600 + dh)
    cfg = config_of(w, flags=flags)
    t = to_dev(with_state(WL.make_inputs(w, with_grads=False), 3, 1e-2), w.io)
    gates = t["q"], t["k"], t["v"], t["eta"], t["beta"], t["gamma"]
    args = *gates, t["w_in"], t["m_in"]
    mats = 2 if fw == 0 else 3
    slot = U * (2 * (mats - 1) + 1) * ((dh + 31) // 32 * 32) * 64 * 2
    assert 256 << 20 < NC * slot
    ref = e2ttt.forward(cfg, *args, save_for_backward=True)[:3]
    assert all(torch.isfinite(r.float()).all() for r in ref)
    *got, ws = e2ttt.forward(cfg, *args)
    assert e2ttt.wait_status(cfg, ws) == 0
    for n, a, b in zip(("out", "w_out", "m_out"), got, ref):
        assert torch.equal(a, b), n
    st = t["w_in"].clone(), t["m_in"].clone()
    out = e2ttt.forward(cfg, *gates, *st, w_out=st[0], m_out=st[1], workspace=ws)[0]
    for n, a, b in zip(("out", "w_out", "m_out"), (out, *st), ref):
        assert torch.equal(a, b), "in place: " + n
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=s):
        e2ttt.forward(cfg, *args, out=got[0], w_out=got[1], m_out=got[2], workspace=ws)
    for _ in range(3):
        for g in got:
            g.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for n, a, b in zip(("out", "w_out", "m_out"), got, ref):
            assert torch.equal(a, b), "graph: " + n
