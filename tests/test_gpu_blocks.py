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
    values (ties), a tile that holds much of what is kept, a gradient that jumps; more than 256 layers.  Most of them are too small for the
    candidate path (test_bounds_that_hold_and_that_fail has those that are not).  Calls without history, around the jump and after it."""
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


def _against_oracle(s, grads, resid, mom, m, ps, ratios, tag):
    after = s.unpack(s.residual)
    u_after = s.unpack(s.momentum_buf) if m is not None else mom
    for l, (blocks, val) in enumerate(s.results()):
        o, u_new = oracle.compress_layer_blocks_momentum(grads[l], mom[l], resid[l], m or 0.0, ps[l], 0.5, ratios[l])
        assert np.array_equal(blocks, o.blocks), (tag, l)
        assert np.array_equal(_bits(val), _bits(np.asarray(o.val).reshape(-1))), (tag, l)
        assert np.array_equal(_bits(after[l]), _bits(o.r_new)), (tag, l)
        if m is not None:
            assert np.array_equal(_bits(u_after[l]), _bits(u_new)), (tag, l)


# grids of block rows by block columns that are large enough for the candidate path: they end on, before and after a tile of 8 by 256, 64 or 32
_GRIDS = {1: [(32, 256), (33, 513), (40, 255), (8, 1025), (72, 129)], 3: [(128, 64), (129, 70), (127, 66), (8, 1030), (64, 130)],
          5: [(256, 128), (257, 129), (255, 130)], 7: [(512, 256), (513, 257)]}


@pytest.mark.parametrize("m, in_place, feed", [(None, False, 0), (None, True, 2), (0.5, False, 2), (0.5, True, 0)],
                         ids=["plain", "in_place_fed", "momentum_fed", "momentum_in_place"])
@pytest.mark.parametrize("sides", [[1], [3], [5], [7], [1, 3, 5]], ids=["p1", "p3", "p5", "p7", "mixed"])
def test_bounds_that_hold_and_that_fail(sides, m, in_place, feed):
    """Every call starts from the same residual (and momentum), so that thresholds settle: two calls without bounds, two on predicted ones, one
    whose gradients are a quarter as large (too few blocks reach the bounds), the calls after it without bounds, one on predicted bounds
    again, one with gradients four times as large (tiles overfill their slots).  Beside the large grids a frozen one, one with
    a tile that holds most of what is kept, a small and a narrow one, one without anything to keep.  The paths are asked for."""
    from paper_2312_17530_amd.session import BlockSession
    large = [(p, r * p - (r + c) % p, c * p - c % p) for p in sides for r, c in _GRIDS[p]]
    p0 = sides[0]
    r0, c0 = _GRIDS[p0][0]
    others = [(p0, r0 * p0, c0 * p0), (p0, r0 * p0, c0 * p0), (p0, 40 * p0, 40 * p0), (p0, 9000 * p0, 2), (p0, r0 * p0, c0 * p0)]
    frozen, hot, none = len(large), len(large) + 1, len(large) + 4
    ps = [x[0] for x in large + others]
    shapes = [x[1:] for x in large + others]
    ratios = [0.02] * (len(shapes) - 1) + [0.0]
    rng = np.random.default_rng(7 + p0 + len(sides))
    s = BlockSession(shapes, 3, 0.5, ratios, ps, in_place=in_place, momentum=m, work_feed=feed)

    def arrays(scale):
        out = [(rng.standard_normal(sh, np.float32) * np.float32(scale)) for sh in shapes]
        out[frozen][:] = 0.0
        out[hot][:8 * p0, :32 * p0] *= np.float32(40.0)
        return out

    resid, mom = arrays(3e-3), arrays(3e-3)
    want = {0: 1, 1: 1, 2: 3, 3: 3, 4: 1, 5: 1, 8: 1, 9: 3, 10: 1}
    for t in range(11):
        scale = 0.25 if 4 <= t <= 9 else 1.0
        grads = arrays(1e-2 * scale)
        r_in, u_in = [[x * np.float32(scale) for x in y] for y in (resid, mom)]
        s.set_grad(grads)
        s.set_residual(r_in)
        if m is not None:
            s.set_momentum(u_in)
        s.compress()
        paths = binding.rsdgc_last_paths_blocks(s.plan, s.workspace)
        if t in want:
            assert paths[:len(large)] == [want[t]] * len(large), t
        assert paths[frozen] == 1 and paths[hot + 1] == 1 and paths[hot + 2] == 1 and paths[none] == 2, t
        if t in (0, 2, 4, 9, 10):
            _against_oracle(s, grads, r_in, u_in if m is not None else [np.zeros(sh, np.float32) for sh in shapes], m, ps, ratios, t)


def test_more_than_4096_chunks():
    """Kept blocks counted beside the ranking, from 33 M blocks on: without bounds, on predicted ones, with failed ones.  Beside the large grid
    ones of more than a million blocks that are all zero and of few values: lists that overflow, scores that tie."""
    from paper_2312_17530_amd.session import BlockSession
    shapes, ratios = [(5800, 5790), (300, 301), (70, 13), (1100, 1000), (1050, 1001)], [0.001, 0.02, 0.1, 0.01, 0.02]
    rng = np.random.default_rng(3)
    s = BlockSession(shapes, 1, 0.5, ratios)
    zero = [np.zeros(sh, np.float32) for sh in shapes]
    for t in range(5):
        grads = [(rng.standard_normal(sh, np.float32) * np.float32(0.25 if t == 4 else 1.0)) for sh in shapes]
        grads[3][:] = 0.0
        grads[4] = rng.integers(-1, 2, shapes[4]).astype(np.float32)
        s.set_grad(grads)
        s.set_residual(zero)
        s.compress()
        paths = binding.rsdgc_last_paths_blocks(s.plan, s.workspace)
        assert paths[:4] == [3 if t in (2, 3) else 1] * 2 + [1, 1], t
        if t in (1, 3, 4):
            _against_oracle(s, grads, zero, zero, None, [1] * 5, ratios, t)
