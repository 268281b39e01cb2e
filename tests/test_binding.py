"""The Python binding's configuration object: what calls derive from it is kept
with it, which must not show in copies, comparisons or pickles."""
import copy
import pickle

from paper_2608_21308_amd import e2ttt


def test_config_copies_and_pickles_after_use():
    cfg = e2ttt.Config(2, 3, 40, 16, 64, 16, e2ttt.FW_SWIGLU, e2ttt.DT_F32)
    before = hash(cfg)
    assert e2ttt.workspace_bytes(cfg, True) > 0       # fills what calls keep
    assert cfg._call[2:] == (2 * 3 * 40 * 16, 2 * 3 * 40, 2 * 3 * cfg.P, 3 * 16)
    for other in (copy.copy(cfg), copy.deepcopy(cfg), pickle.loads(pickle.dumps(cfg))):
        assert other == cfg and hash(other) == before
        assert e2ttt.workspace_bytes(other, True) == e2ttt.workspace_bytes(cfg, True)
