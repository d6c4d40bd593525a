"""The block reading over many calls: candidates against predicted bounds, layers that stay on the full score map, bounds that fail in the
middle of a training and tiles that overfill their slots, against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2312_17530_amd import binding

pytestmark = pytest.mark.gpu


def _bits(a):
    return np.ascontiguousarray(a, dtype=np.float32).view(np.uint32)


@pytest.mark.parametrize("m, in_place, feed, more", [(None, False, 0, 0), (None, True, 2, 0), (0.9, False, 2, 0), (0.9, True, 0, 0), (None, True, 0, 300)],
                         ids=["plain", "in_place_fed", "momentum_fed", "momentum_in_place", "many_layers"])
@pytest.mark.parametrize("sides", [[1], [3], [5], [7], [1, 3, 5, 7]], ids=["p1", "p3", "p5", "p7", "mixed"])
def test_blocks_call_after_call(sides, m, in_place, feed, more):
    """Grids that end on, before and after a tile of 8 by 32, 64 or 256 blocks, one tile and several, rows of odd length and grids cut by the
    matrix's edges; narrow grids and ratios beyond the candidate path's (full map), one without anything to keep, frozen ones (no bound), few
    values (ties), a tile that overfills its slot, a gradient that jumps; more than 256 layers.  Calls without history, on
    predicted bounds, around the jump and after it."""
    from paper_2312_17530_amd.session import BlockSession
    p0 = max(sides)
    shapes = [(8 * p0, 64 * p0), (16 * p0 + 1, 130 * p0 + 2), (24 * p0 - 1, 257 * p0), (9 * p0, 33 * p0 + 1), (40, 40), (300, 5), (17 * p0, 70 * p0),
              (20 * p0, 90 * p0), (16 * p0, 128 * p0 - 3), (32 * p0, 300 * p0 + 5), (1, 700), (40 * p0, 64 * p0)]
    ratios = [0.02, 0.03, 0.02, 0.05, 0.05, 0.05, 0.5, 0.0, 0.02, 0.01, 0.02, 0.03]
    frozen, tied, hot = {8}, {1}, 11
    if p0 <= 3 and m is None:                          # (rows so long that the gather counts by row)
        shapes, ratios = shapes + [(12 * p0, 33000 * p0)], ratios + [0.02]
    shapes, ratios = shapes + [(1 + l % 5, 1 + l % 70) for l in range(more)], ratios + [(0.0, 1.0, 0.3)[l % 3] for l in range(more)]
    ps = [sides[l % len(sides)] for l in range(len(shapes))]
    rng = np.random.default_rng(90 + sides[0] + len(sides))
    s = BlockSession(shapes, 3, 0.5, ratios, ps, in_place=in_place, momentum=m, work_feed=feed)
    for t in range(12):
        scale = 10.0 if t == 9 else 1e-2
        grads = [np.zeros(sh, np.float32) if l in frozen else (rng.integers(-1, 2, sh) * scale).astype(np.float32) if l in tied else
                 (rng.standard_normal(sh) * scale).astype(np.float32) for l, sh in enumerate(shapes)]
        grads[hot][:8 * ps[hot], :30 * ps[hot]] *= np.float32(30.0 if t != 5 else 1.0)
        resid = s.unpack(s.residual)
        mom = s.unpack(s.momentum_buf) if m is not None else [np.zeros(sh, np.float32) for sh in shapes]
        s.set_grad(grads)
        s.compress()
        if t in (3, 4, 6):
            continue
        after = s.unpack(s.residual)
        u_after = s.unpack(s.momentum_buf) if m is not None else mom
        for l, (blocks, val) in enumerate(s.results()):
            o, u_new = oracle.compress_layer_blocks_momentum(grads[l], mom[l], resid[l], m or 0.0, ps[l], 0.5, ratios[l])
            assert np.array_equal(blocks, o.blocks), (t, l)
            assert np.array_equal(_bits(val), _bits(np.asarray(o.val).reshape(-1))), (t, l)
            assert np.array_equal(_bits(after[l]), _bits(o.r_new)), (t, l)
            if m is not None:
                assert np.array_equal(_bits(u_after[l]), _bits(u_new)), (t, l)
