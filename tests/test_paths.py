"""Which kernels a call takes (CPU; read off the buffer sizes): calls timed on both
paths go to the faster one, saving or not, and the two kinds of a call may share
a saving workspace whatever their paths."""
import pytest

from paper_2608_21308_amd import e2ttt
from tests.path_util import query_apart, takes_tiles

MLP, SWIGLU = e2ttt.FW_MLP, e2ttt.FW_SWIGLU


def cfg(fw, d, dh, U, T, C, flags=0):
    return e2ttt.Config(B=1, H=U, T=T, d=d, dh=dh, chunk=C, fw=fw, io=e2ttt.DT_BF16, flags=flags)


# chain time over tiles time, forward and training step, as measured
@pytest.mark.parametrize("fw,d,dh,U,T,C,fwd,step", [
    (MLP, 128, 33, 107, 69, 68, 0.86, 0.92),       # narrow nets of many units
    (MLP, 128, 64, 128, 350, 100, 0.93, 0.94),
    (MLP, 128, 33, 356, 294, 70, 0.70, 0.70),      # more units than workgroups at once
    (MLP, 64, 168, 311, 391, 391, 0.89, 0.82),
    (SWIGLU, 64, 158, 413, 255, 102, 0.80, 0.90),
    (MLP, 64, 120, 64, 448, 128, 0.91, 0.96),
    (SWIGLU, 64, 118, 80, 187, 75, 0.92, None),
    (MLP, 64, 256, 128, 448, 128, 0.5, 0.6),
    (MLP, 64, 256, 8, 448, 128, 1.3, 1.5),
    (MLP, 64, 256, 32, 1792, 512, 2.1, 2.2),
    (MLP, 128, 512, 8, 448, 128, 2.0, 2.2),
    (MLP, 128, 512, 32, 2048, 512, 2.5, 2.5),
    (MLP, 128, 512, 128, 448, 128, 1.5, 1.6),
    (SWIGLU, 128, 344, 16, 1500, 512, 4.9, 4.9),
])
def test_the_faster_path_is_taken(fw, d, dh, U, T, C, fwd, step):
    c = cfg(fw, d, dh, U, T, C)
    assert takes_tiles(c, False) == (fwd > 1.0)
    if step is not None:
        assert takes_tiles(c, True) == (step > 1.0)


def test_what_never_takes_the_tiles():
    assert not takes_tiles(cfg(MLP, 128, 512, 8, 640, 64), False)            # up to 64 tokens
    assert not takes_tiles(cfg(MLP, 128, 512, 8, 60, 512), True)
    assert not takes_tiles(cfg(SWIGLU, 128, 400, 8, 1024, 512), True)        # too wide for LDS
    assert not takes_tiles(cfg(MLP, 64, 256, 8, 448, 128, e2ttt.FLAG_POST_NORM), True)


def test_query_side_apart_where_few_units_have_chunks_enough():
    assert query_apart(cfg(MLP, 64, 256, 32, 512, 64))
    assert not query_apart(cfg(MLP, 64, 256, 33, 512, 64))
    assert not query_apart(cfg(MLP, 64, 256, 32, 448, 64))
    assert query_apart(cfg(MLP, 64, 128, 64, 512, 64))
    assert not query_apart(cfg(MLP, 128, 256, 8, 512, 64))


def test_a_saving_workspace_serves_either_call():
    n = 0
    for fw, dhs in ((MLP, (48, 120, 256)), (SWIGLU, (64, 118, 172))):
        for dh in dhs:
            for U in range(1, 130, 3):
                for C in (65, 75, 100, 128, 300):
                    c = cfg(fw, 64, dh, U, 5 * C // 2, C)
                    assert e2ttt.workspace_bytes(c, True) >= e2ttt.workspace_bytes(c, False)
                    n += takes_tiles(c, True) != takes_tiles(c, False)
    assert n > 0      # (calls whose saving and other kind differ are among them)
