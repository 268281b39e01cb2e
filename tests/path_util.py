"""Which kernels a call takes, read off the library's buffer sizes (no GPU).

The post-chunk normalisation always runs on the chain kernels, and what it adds
to a chain call's buffers is known; a call whose buffers differ from those of
the same call with the normalisation by anything else takes the token-tiled
path.  A backward of a chain that leaves its query side out has that side's
operands in its scratch."""
import dataclasses

from paper_2608_21308_amd import e2ttt


def align(n):
    return (n + 255) // 256 * 256


def groups(cfg):
    """Workgroups per unit of the chain kernels."""
    nblk = (cfg.dh + 15) // 16
    if cfg.io != e2ttt.DT_BF16:
        return 1
    if cfg.d == 128:
        widths = (4, 8, 16, 24, 32) if cfg.fw == e2ttt.FW_SWIGLU else (4, 8, 16, 32)
        ns = (1, 2, 4, 6, 8) if cfg.fw == e2ttt.FW_SWIGLU else (1, 2, 4, 8)
    elif cfg.fw == e2ttt.FW_MLP:
        widths, ns = (8, 16), (1, 2)
    else:
        widths, ns = (4, 8, 12), (1, 2, 3)
    return next(n for w, n in zip(widths, ns) if nblk <= w)


def takes_tiles(cfg, saving):
    """Token-tiled path, of a call that saves for the backward or does not."""
    if cfg.flags & e2ttt.FLAG_POST_NORM:
        return False
    pn = dataclasses.replace(cfg, flags=cfg.flags | e2ttt.FLAG_POST_NORM)
    U, ns = cfg.B * cfg.H, groups(cfg)
    rows = (1 if cfg.fw == e2ttt.FW_MLP else 2) * cfg.dh + cfg.d
    xchg = align(max(min((U + 7) // 8 * 8, 128) if ns > 1 else 0, 1) * ns * 2 * cfg.d * 4)
    if saving:
        diff = e2ttt.backward_scratch_bytes(pn) - e2ttt.backward_scratch_bytes(cfg)
        return diff != align(U * ns * rows * 4) + xchg
    diff = e2ttt.workspace_bytes(pn, False) - e2ttt.workspace_bytes(cfg, False)
    return diff != align(U * rows * 4) + xchg


def query_apart(cfg):
    """Chain whose saving forward and backward leave the query side out: its
    operands, of every 32-token tile, outweigh the rest of the scratch by far."""
    if cfg.io != e2ttt.DT_BF16 or cfg.d != 64 or takes_tiles(cfg, True):
        return False
    tiles = cfg.B * cfg.H * cfg.n_chunks * ((min(cfg.chunk, cfg.T) + 31) // 32)
    mats = 2 if cfg.fw == e2ttt.FW_MLP else 3
    return cfg.n_chunks >= 8 and e2ttt.backward_scratch_bytes(cfg) >= \
        tiles * (2 * (cfg.d // 16) + mats * ((cfg.dh + 31) // 32 * 2)) * 1024
