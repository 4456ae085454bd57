"""Lazy calls that walk in several passes: the shapes, shared by the GPU tests
and by the test (on the host stand-in) that these shapes do walk, and the
oracle's lazy results from its eager statistics.

Whether a call walks depends on what a pass over W_U costs, so a shape that
walks needs a matrix and a number of positions of some size: too large for the
oracle's lazy projection, which projects one position at a time."""
import numpy as np

import oracle as O

# name, K, B, n per sequence, d, V, dtype, every position walks, normalized, exact ties
WALKS = [
    # counts on the device: passes in the size classes <= 64, <= 128, <= 192 and above, over one and several layers
    ("band", 4, 1, 200, 2048, 30011, "bf16", False, False, False),
    ("band_norm", 4, 1, 200, 2048, 30011, "bf16", False, True, False),
    ("band_8_layers", 8, 1, 250, 2048, 20011, "bf16", False, False, False),
    ("all_classes", 5, 1, 230, 2048, 60013, "bf16", True, False, False),
    # more layers than a reduction has waves, and the most the boundary takes: passes of 2, 4, .. layers at least
    ("band_13_layers", 13, 1, 60, 2048, 30011, "bf16", False, False, False),
    ("band_64_layers", 64, 1, 20, 2048, 30011, "bf16", False, False, False),
    # 2000 rows at most, far fewer in truth
    ("all_13_layers", 13, 1, 250, 2048, 20011, "bf16", True, False, False),
    # above 256 positions: counts waited for, then on the device
    ("readback", 5, 2, 150, 2048, 60013, "bf16", True, False, False),
    ("readback_norm", 4, 3, 200, 2048, 20011, "bf16", True, True, False),
    # tied tops: the reduction of a pass resolves them for the forms whose tiles sum in orders of their own
    ("ties_near", 36, 1, 25, 2048, 30011, "bf16", False, False, "near"),
    ("ties_far", 8, 1, 250, 2048, 20011, "bf16", False, False, "far"),
    ("ties_readback", 4, 2, 300, 2048, 20011, "bf16", True, False, "far"),
    ("f32_all", 4, 1, 160, 2048, 30011, "f32", True, False, False),
    ("f32_13_layers", 13, 1, 60, 2048, 10007, "f32", True, False, False),
    ("f32_readback", 5, 2, 150, 2048, 10007, "f32", True, False, False),
    ("f32_band_norm", 4, 1, 200, 2048, 4003, "f32", False, True, False),
]


def stop_early(w, seed):
    """Let each masked position agree on a drawn number of layers below the
    final one (0 .. K - 1): below them it has another position's states."""
    g = np.random.default_rng(seed)
    K = w.cfg.K
    pos = np.array(O.masked_positions(w.mask))
    keep = g.integers(0, K, size=len(pos))
    other = np.roll(pos, 1, axis=0)
    for l in range(K - 1):
        cut = K - 1 - l > keep
        rows = w.hidden[l, other[cut, 0], other[cut, 1]]   # a copy, taken before any is replaced
        w.hidden[l, pos[cut, 0], pos[cut, 1]] = rows


def lazy_from_eager(mask, pos, layer, P):
    """What O.score_commit_lazy returns, from the eager statistics of every
    layer (O.layer_stats_masked): the layers that a walk does not come to are
    taken out."""
    y = layer["argmax"]
    n, K = y.shape
    c = layer["conf"][:, K - 1]
    walks = ~np.isnan(c) if P.lazy_all else (c >= P.theta_c) & (c < P.theta_h)
    suffix = 1 + np.cumprod(y[:, -2::-1] == y[:, -1:], axis=1).sum(1) if K > 1 else np.ones(n, np.int64)
    depth = np.where(walks, np.minimum(suffix + 1, K), 1)
    unseen = np.arange(K)[None, :] < (K - depth)[:, None]
    lay = {k: np.where(unseen, -1 if k == "argmax" else np.nan, v) for k, v in layer.items()}
    o = O.assemble(mask, pos, lay, P)
    for (b, i), v in zip(pos, walks):
        if not v:
            o["persistence"][b, i] = -1
            o["drop"][b, i] = o["stability"][b, i] = np.nan
    o["layers_projected"] = depth
    return o
