"""Workspace sizes of the chains that leave the query side out (CPU): operand
copies of every chunk are saved up to 16 GiB of them; above, a saving call's
workspace and scratch are the chain's own again, while a call without saving
keeps a bounded number of chunks' copies."""
import pytest

from paper_2608_21308_amd import e2ttt

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
