"""The token-tiled path of long chunks (csrc/tile_fwd.hip, tile_bwd.hip) at the
sizes where it can go wrong: a last tile of one token, chunks just over one
tile of the chain kernels, a ragged last chunk shorter than a tile, hidden
widths that are no multiple of 32 or 128 (waves without a block), both sides
of the unit count where workgroups are laid out per XCD, initial momentum and
state gradients.  Each shape is one that the path takes; the bar is that of the
other bf16 tests (2e-2 against the fp64 oracle, with the local maxima)."""
import numpy as np
import pytest
import torch

from paper_2608_21308_amd import e2ttt, workloads as WL
from tests.gpu_util import TOL, config_of, to_dev
from tests.path_util import takes_tiles
from tests.test_gpu_backward import errors as berrors, gpu_fwd_bwd, oracle_bwd, with_state_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fw,d,dh,B,H,T,C,flags", [
    (0, 64, 256, 1, 2, 65, 65, 0),      # one chunk, a last tile of one token
    (0, 64, 40, 1, 3, 300, 97, 0),      # dh just over one block of 32, last chunk of nine tokens
    (0, 64, 250, 3, 3, 200, 66, 0),     # nine units: one on a second round of the XCDs
    (1, 64, 172, 1, 2, 261, 130, 1),    # SwiGLU, a last chunk of one token
    (1, 64, 64, 2, 4, 150, 75, 1),
    (0, 128, 512, 1, 2, 520, 512, 0),   # the widest net, a last chunk of eight tokens
    (0, 128, 130, 1, 1, 97, 96, 0),
    (1, 128, 344, 1, 2, 160, 128, 1),
    (1, 128, 384, 1, 9, 130, 129, 1),   # the widest SwiGLU of the path
])
def test_tiles_forward_backward(fw, d, dh, B, H, T, C, flags):
    w = WL.WORKLOADS[1].with_(fw=fw, B=B, H=H, T=T, d=d, dh=dh, C=C, backward=True,
                              seed=4100 + T + dh)
    assert takes_tiles(config_of(w, flags=flags), True)
    x = with_state_inputs(WL.make_inputs(w), 5, 1e-2)
    errs = berrors(gpu_fwd_bwd(w, x, flags), oracle_bwd(w, x, flags), C=C)
    print("tiles fw=%d d=%d dh=%d U=%d T=%d C=%d" % (fw, d, dh, B * H, T, C),
          {k: "%.2e" % v for k, v in errs.items()}, flush=True)
    assert all(e <= TOL["bf16"] for e in errs.values()), errs


def test_static_workspace_too_small_for_tiles_runs_the_chain():
    # the token-tiled path would need more than the library's array for these
    # units; the call is still accepted and agrees with the path's own results
    # to the rounding of the two summation orders
    w = WL.WORKLOADS[1].with_(B=4, H=16, T=150, d=128, dh=512, C=150, seed=4200)
    cfg = config_of(w)
    assert e2ttt.workspace_bytes(cfg, False) > e2ttt.STATIC_WORKSPACE_BYTES
    t = to_dev(WL.make_inputs(w, with_grads=False), w.io)
    args = t["q"], t["k"], t["v"], t["eta"], t["beta"], t["gamma"], t["w_in"], None
    ref = e2ttt.forward(cfg, *args)[:3]
    got = tuple(torch.full_like(r, float("nan")) for r in ref)
    e2ttt.forward_static(cfg, *args, *got)
    for n, a, b in zip(("out", "w_out", "m_out"), got, ref):
        a, b = a.float().cpu().numpy(), b.float().cpu().numpy()
        assert np.linalg.norm(a - b) <= 1e-2 * np.linalg.norm(b), n


def test_first_layer_deltas_are_whole():
    # with W1 = 0 the net's output, its LayerNorm row and dY are the same numbers
    # on both paths (no rounding to bf16 can fall the other way), and dH = dY W2 / 2
    # differs by the order of its fp32 sum at most.  The state sums then agree to
    # fp32 rounding: 150 terms of 2^-24 with random signs, 8e-7 at most (measured
    # 0).  dH rounded to two bf16 parts on its way through memory gave 3.2e-6.
    w = WL.WORKLOADS[1].with_(B=4, H=16, T=150, d=128, dh=512, C=150, seed=4250)
    cfg = config_of(w)
    assert e2ttt.workspace_bytes(cfg, False) > e2ttt.STATIC_WORKSPACE_BYTES   # (static: the chain)
    x = WL.make_inputs(w)
    x["w_in"][..., :512 * 128] = 0.0
    t = to_dev(x, w.io)
    args = t["q"], t["k"], t["v"], t["eta"], t["beta"], t["gamma"], t["w_in"], None
    tiles = e2ttt.forward(cfg, *args)[1:3]
    chain = [torch.empty_like(r) for r in tiles]
    e2ttt.forward_static(cfg, *args, torch.empty_like(t["q"]), *chain)
    for n, a, b in zip(("w_out", "m_out"), tiles, chain):
        a, b = a[..., :512 * 128].double(), b[..., :512 * 128].double()
        err = float((a - b).norm() / b.norm())
        print("first layer", n, "%.2e" % err, flush=True)
        assert err <= 8e-7, (n, err)


def test_saving_and_other_calls_on_different_paths_share_a_workspace():
    # a shape whose saving call takes the one path and whose other call the other:
    # on one buffer in turn, each reports its own status and both agree to the
    # rounding of the two summation orders
    cfgs = (e2ttt.Config(B=1, H=U, T=5 * C // 2, d=64, dh=dh, chunk=C, fw=fw, io=e2ttt.DT_BF16)
            for fw, dh in ((0, 256), (1, 172)) for U in range(8, 130, 8) for C in (75, 100, 128, 300))
    cfg = next(c for c in cfgs if takes_tiles(c, True) != takes_tiles(c, False))
    w = WL.WORKLOADS[1].with_(fw=cfg.fw, B=1, H=cfg.H, T=cfg.T, d=64, dh=cfg.dh, C=cfg.chunk,
                              backward=True, seed=4260)
    t = to_dev(WL.make_inputs(w, with_grads=True), w.io)
    args = t["q"], t["k"], t["v"], t["eta"], t["beta"], t["gamma"], t["w_in"], None
    ws = e2ttt.alloc_workspace(cfg, True)
    scratch = torch.empty(e2ttt.backward_scratch_bytes(cfg), dtype=torch.uint8, device="cuda")
    ws.fill_(255)
    scratch.fill_(255)
    outs = []
    for saving in (False, True, False):
        outs.append(e2ttt.forward(cfg, *args, workspace=ws, save_for_backward=saving)[:3])
        assert e2ttt.wait_status(cfg, ws) == 0
        if saving:
            e2ttt.backward(cfg, *args, ws, t["d_out"], scratch=scratch)
            assert e2ttt.wait_status(cfg, ws, scratch) == 0
    for a, b, c in zip(*outs):
        assert torch.equal(a, c)
        a, b = a.double(), b.double()
        assert float((a - b).norm()) <= 1e-2 * float(b.norm())


def test_state_in_place_and_under_capture():
    # w_out over w_in, m_out over m_in; and the launches of all chunks as one graph
    w = WL.WORKLOADS[1].with_(fw=0, B=1, H=3, T=300, d=64, dh=256, C=97, seed=4270)
    cfg = config_of(w)
    assert takes_tiles(cfg, False)
    x = with_state_inputs(WL.make_inputs(w, with_grads=False), 5, 1e-2, False)
    t = to_dev(x, w.io)
    args = t["q"], t["k"], t["v"], t["eta"], t["beta"], t["gamma"]
    *ref, ws = e2ttt.forward(cfg, *args, t["w_in"], t["m_in"])
    st = t["w_in"].clone(), t["m_in"].clone()
    out = e2ttt.forward(cfg, *args, *st, w_out=st[0], m_out=st[1], workspace=ws)[0]
    for n, a, b in zip(("out", "w_out", "m_out"), (out, *st), ref):
        assert torch.equal(a, b), n
    got = [torch.empty_like(r) for r in ref]
    s, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=s):
        e2ttt.forward(cfg, *args, t["w_in"], t["m_in"], out=got[0], w_out=got[1], m_out=got[2],
                      workspace=ws)
    for _ in range(3):
        for g in got:
            g.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for n, a, b in zip(("out", "w_out", "m_out"), got, ref):
            assert torch.equal(a, b), "graph: " + n
