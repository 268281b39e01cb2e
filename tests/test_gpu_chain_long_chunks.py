"""Chunks longer than the token tile where they stay on the chain kernels (head dim
64, bf16: many units, or units enough for the chain to be the faster path), with
the query side in the chain and apart, against the fp64 oracle on sampled units;
and non-finite values on the token-tiled path and beside a chain that leaves its
query side out.  Every case asserts the path it is there for."""
import numpy as np
import pytest
import torch

from paper_2608_21308_amd import e2ttt, workloads as WL
from tests import fp32ref
from tests.gpu_util import TOL, config_of
from tests.path_util import query_apart, takes_tiles
from tests.test_gpu_nonfinite import GRADS, same_mask_and_close, spoil
from tests.test_gpu_post_norm import errors, run_gpu, run_oracle, with_state

pytestmark = pytest.mark.gpu

BARE = e2ttt.FLAG_NO_RESIDUAL_LN


def sampled(w, flags, backward=True):
    """Errors of the first, a middle and the last unit, and the gate gradients' bars."""
    x = with_state(WL.make_inputs(w, with_grads=True), 7, 1e-2)
    U = w.B * w.H
    units = [0, U // 2 + 1, U - 1]

    def pick(a):
        return a if a is None else np.ascontiguousarray(a.reshape((U,) + a.shape[2:])[units][None])

    got = {n: pick(a) for n, a in run_gpu(w, x, flags, backward=backward).items()}
    xs = {n: pick(a) for n, a in x.items()}
    ref = run_oracle(w, xs, flags)
    errs = errors(got, {n: r for n, r in ref.items() if n in got}, xs, w.C)
    if not backward:
        return errs, {}
    return errs, fp32ref.bf16_state_bar(errors, xs, ref, C=w.C, fw=w.fw, dh=w.dh, flags=flags)


def check(errs, bar, what):
    print(what, "worst %.2e %s" % max((e, n) for n, e in errs.items()),
          {n: "%.1e" % b for n, b in bar.items() if b > TOL["bf16"]}, flush=True)
    assert all(e <= bar.get(n, TOL["bf16"]) for n, e in errs.items()), (what, errs)


@pytest.mark.parametrize("fw,dh,B,H,T,C,flags", [
    (0, 256, 8, 16, 1100, 512, 0),     # two workgroups per unit, a last chunk of two tiles
    (0, 250, 4, 16, 237, 80, 0),       # three chunks, tiles of 64 and 16 tokens
    (0, 120, 6, 16, 250, 100, 0),      # one workgroup of eight waves
    (0, 64, 8, 16, 131, 65, 0),        # a tile and a chunk of one token
    (1, 172, 8, 16, 300, 128, BARE),   # SwiGLU: W_0 from its block after the first tile
    (1, 128, 8, 16, 300, 130, BARE),
    (1, 64, 8, 16, 66, 65, 0),
    (1, 172, 8, 16, 131, 128, 0),      # with the residual LayerNorm
])
def test_long_chunks_on_the_chain(fw, dh, B, H, T, C, flags):
    w = WL.WORKLOADS[1].with_(fw=fw, B=B, H=H, T=T, d=64, dh=dh, C=C, backward=True,
                              seed=4700 + T + dh)
    cfg = config_of(w, flags=flags)
    assert not takes_tiles(cfg, True) and not query_apart(cfg)
    what = "chain fw=%d dh=%d U=%d T=%d C=%d" % (fw, dh, B * H, T, C)
    check(*sampled(w, flags), what)
    if not takes_tiles(cfg, False):
        check(*sampled(w, flags, backward=False), what + " (not saving)")


@pytest.mark.parametrize("fw,dh,U,T,C,flags,saving", [
    (0, 120, 48, 1100, 128, 0, True),          # nine chunks of two tiles, the last shorter
    (0, 60, 64, 1025, 128, BARE, True),        # a last chunk of one token
    (0, 120, 48, 1100, 128, 0, False),
    (1, 62, 25, 946, 114, BARE, False),        # SwiGLU
    (0, 206, 19, 5922, 99, BARE, False),       # two workgroups, 60 chunks
])
def test_long_chunks_with_the_query_side_apart(fw, dh, U, T, C, flags, saving):
    w = WL.WORKLOADS[1].with_(fw=fw, B=1, H=U, T=T, d=64, dh=dh, C=C, backward=True,
                              seed=4800 + T + dh)
    cfg = config_of(w, flags=flags)
    assert not takes_tiles(cfg, saving) and cfg.n_chunks >= 8
    assert not saving or query_apart(cfg)
    check(*sampled(w, flags, backward=saving),
          "apart fw=%d dh=%d U=%d T=%d C=%d saving=%d" % (fw, dh, U, T, C, saving))


# one value of one unit: which elements become non-finite, and the others' values
@pytest.mark.parametrize("where", ["q", "k", "v", "eta", "d_out"])
@pytest.mark.parametrize("fw,d,dh,T,C,flags", [
    (0, 64, 256, 200, 80, 0), (1, 64, 172, 130, 75, 0), (0, 128, 200, 200, 80, 0),   # tiles
    (0, 64, 256, 129, 16, 0), (1, 64, 172, 130, 16, BARE)])                          # apart
def test_nonfinite_on_tiles_and_apart(where, fw, d, dh, T, C, flags):
    w = WL.WORKLOADS[1].with_(fw=fw, B=1, H=2, T=T, d=d, dh=dh, C=C, backward=True, seed=4900 + dh)
    cfg = config_of(w, flags=flags)
    assert takes_tiles(cfg, True) if C > 64 else query_apart(cfg)
    x = spoil(WL.make_inputs(w), where, np.nan)
    ref, got = run_oracle(w, x, flags), run_gpu(w, x, flags)
    free = run_gpu(w, x, flags, backward=False)
    n = 0
    for name in ("out", "w_out", "m_out") + GRADS:
        block = None if name in ("w_out", "m_out", "d_w_in", "d_m_in") else min(C, 64)
        n += same_mask_and_close(torch.from_numpy(got[name]), ref[name], name, TOL["bf16"], block)
        if name in free:
            same_mask_and_close(torch.from_numpy(free[name]), ref[name], name, TOL["bf16"], block)
    assert n > 0
