"""Workspace sizes of the chains that leave the query side out (CPU): operand
copies of every chunk are saved up to 16 GiB of them; above, a saving call's
workspace and scratch are the chain's own again, while a call without saving
keeps a bounded number of chunks' copies.  The same bound for the token-tiled
path, and for the operands in the backward's scratch."""
import dataclasses

import pytest

from paper_2608_21308_amd import e2ttt
from tests.path_util import takes_tiles

GIB = 1 << 30


def sizes(fw, dh, U, T):
    cfg = e2ttt.Config(B=1, H=U, T=T, d=64, dh=dh, chunk=64, fw=fw, io=e2ttt.DT_BF16)
    return (e2ttt.workspace_bytes(cfg, False), e2ttt.workspace_bytes(cfg, True),
            e2ttt.backward_scratch_bytes(cfg))


@pytest.mark.parametrize("fw,dh,U", [(0, 128, 64), (0, 256, 16), (1, 172, 32)])
def test_saved_copies_are_bounded(fw, dh, U):
    mats = 2 if fw == 0 else 3
    slot = U * 3 * mats * ((dh + 31) // 32 * 32) * 64 * 2     # one chunk's copies
    last = 16 * GIB // slot                                    # chunks that still fit
    below, above = sizes(fw, dh, U, 64 * last), sizes(fw, dh, U, 64 * (last + 1))
    assert below[1] > 16 * GIB - slot and above[1] < below[1]
    assert above[2] < below[2] // 8                            # (the query's operands)
    assert above[0] - below[0] < GIB // 4                      # without saving: alike


def slot_bytes(fw, dh, U):
    # one chunk's copies without saving
    mats = 2 if fw == 0 else 3
    return U * (2 * (mats - 1) + 1) * ((dh + 31) // 32 * 32) * 64 * 2


@pytest.mark.parametrize("fw,dh,U,NC", [(0, 256, 8, 13), (0, 256, 8, 32), (0, 256, 32, 64),
                                        (1, 172, 8, 64), (1, 172, 16, 128), (0, 120, 64, 40)])
def test_one_launch_where_the_copies_fit(fw, dh, U, NC):
    # (a launch too many costs as much as the query sides of some twenty chunks)
    slot = slot_bytes(fw, dh, U)
    assert NC * slot <= 256 << 20
    assert sizes(fw, dh, U, 64 * NC)[0] - sizes(fw, dh, U, 64 * 8)[0] >= (NC - 8) * slot


@pytest.mark.parametrize("fw,dh,U", [(0, 256, 8), (1, 172, 16), (0, 120, 64), (1, 64, 2)])
@pytest.mark.parametrize("T", [512, 2048, 8192])
def test_buffers_serve_other_calls_up_to_64_mb(fw, dh, U, T):
    # a backward's scratch a forward without saving; a buffer for long chunks the same
    # tokens in chunks of 64
    free, _, scratch = sizes(fw, dh, U, T)
    assert scratch >= min(free, 64 << 20)
    for C in (128, 512):
        long = e2ttt.Config(B=1, H=U, T=T, d=64, dh=dh, chunk=C, fw=fw, io=e2ttt.DT_BF16)
        if takes_tiles(long, False):
            assert e2ttt.workspace_bytes(long, False) >= min(free, 64 << 20)
        if takes_tiles(long, True):
            assert e2ttt.backward_scratch_bytes(long) >= min(scratch, 64 << 20)


def need(cfg):
    return e2ttt.workspace_bytes(cfg, True) + e2ttt.backward_scratch_bytes(cfg)


@pytest.mark.parametrize("fw,d,dh,U,T,C", [(0, 128, 512, 4, 20, 512), (0, 64, 256, 4, 20, 512),
                                           (1, 64, 172, 8, 20, 512), (0, 128, 512, 8, 18, 65),
                                           (0, 64, 120, 16, 21, 80), (1, 128, 344, 2, 20, 72),
                                           (0, 64, 120, 64, 19, 512), (0, 64, 120, 2, 17, 1)])
@pytest.mark.parametrize("flags", [0, e2ttt.FLAG_POST_NORM])
def test_long_sequences_need_little_more_than_on_the_chain(fw, d, dh, U, T, C, flags):
    cfg = e2ttt.Config(B=1, H=U, T=1 << T, d=d, dh=dh, chunk=C, fw=fw, io=e2ttt.DT_BF16, flags=flags)
    # the chain's saved state in the operand type, LayerNorm rows and (MLP) the
    # query side's activations and derivatives, as of one chunk of the bare chain:
    # too few chunks to leave the query side out, too short for the token-tiled path
    few = dataclasses.replace(cfg, T=4 * C, flags=cfg.flags | e2ttt.FLAG_POST_NORM)
    chain = need(few) * (cfg.n_chunks / 4.0)
    assert need(cfg) <= max(1.1 * chain, 33 * GIB)
    if takes_tiles(cfg, True):      # its scratch: one chunk's operands, 64 MB, the scalar kernels'
        assert e2ttt.backward_scratch_bytes(cfg) <= GIB // 8 + 16 * U * cfg.T
