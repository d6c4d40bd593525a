"""The residual's own arena takes v while the scores are formed (rsdgc_compress with residual_out == residual, plans that do not
select in one launch): windows inside a tile by the main pass, those across its edges by the pass that follows, against the
oracle."""
import numpy as np
import pytest

import oracle
from paper_2312_17530_amd import binding

pytestmark = pytest.mark.gpu


def _bits(a):
    return np.ascontiguousarray(a, dtype=np.float32).view(np.uint32)


@pytest.mark.parametrize("sides, more, feed", [([1], 0, 0), ([1], 0, 2), ([1], 4100, 0), ([3], 0, 2), ([3], 4100, 2), ([3], -1, 0), ([5], 0, 2), ([7], 0, 2),
                                               ([1, 3, 5, 7], 0, 2), ([1, 3, 5, 3], -1, 0), ([7], 0, 0), ([1, 3], 4100, 0)])
def test_one_arena(sides, more, feed):
    """Matrices that end on, before and after a tile's 16 rows and 256 columns, within a window's reach of them, one tile high or
    wide, rows of odd length; a layer always ranked on the full map (whose v is formed when it is marked), one without
    anything to keep, frozen ones (no bound), few values (ties), a tile that overfills its slot; then a gradient that jumps, so that
    bounds fail after v has replaced the residual.  Calls without history, on predicted bounds and around the jump.  Plans that v replaces the
    residual in because of their size (more < 0: a large layer without anything to keep) or their single elements, by both forms of the
    emit; the others, with and without the work feed, that it does not."""
    from paper_2312_17530_amd.session import Session
    shapes = [(40, 40), (33, 512), (16, 256), (17, 257), (48, 768), (18, 259), (35, 1030), (15, 511), (64, 27), (1, 700), (3, 2100),
              (130, 131), (49, 1028), (32, 513), (50, 64), (34, 300), (64, 520)]
    ratios = [0.9, 0.02, 0.02, 0.05, 0.03, 0.05, 0.02, 0.05, 0.03, 0.02, 0.02, 0.04, 0.01, 0.05, 0.0, 0.02, 0.02]
    frozen, tied, hot = {13}, {15}, 16
    if more < 0:
        shapes, ratios = shapes + [(4096, 8200)], ratios + [0.0]
    shapes, ratios = shapes + [(1, 1 + l % 70) for l in range(more)], ratios + [(0.0, 1.0, 0.3)[l % 3] for l in range(more)]
    ps = [sides[l % len(sides)] for l in range(len(shapes))]
    rng = np.random.default_rng(70 + sides[0] + len(sides))
    s = Session(shapes, 3, 0.5, ratios, ps, in_place=True, work_feed=feed)
    failed = set()
    for t in range(15 if more <= 0 else 3):
        scale = 10.0 if t == 13 else 1e-2
        grads = [np.zeros(sh, np.float32) if l in frozen else (rng.integers(-1, 2, sh) * scale).astype(np.float32) if l in tied else
                 (rng.standard_normal(sh, np.float32) * np.float32(scale)) for l, sh in enumerate(shapes)]
        grads[hot][16:32, :256] *= np.float32(30.0)
        resid = s.unpack(s.residual)
        s.set_grad(grads)
        s.compress()
        if t == 13:
            failed = {l for l, x in enumerate(binding.rsdgc_last_paths(s.plan, s.workspace)) if x == 1}
        if 2 <= t < 11:
            continue
        after = s.unpack(s.residual)
        for l, (idx, val, centres, _) in enumerate(s.results()):
            if ratios[l] == 0.0 and grads[l].size > 1 << 20:
                assert len(idx) == 0 and np.array_equal(_bits(after[l]), _bits(resid[l] + grads[l])), t
                continue
            o = oracle.compress_layer(grads[l], resid[l], ps[l], 0.5, ratios[l])
            assert np.array_equal(idx, o.idx) and np.array_equal(centres, o.centres), (t, l)
            assert np.array_equal(_bits(val), _bits(o.val)) and np.array_equal(_bits(after[l]), _bits(o.r_new)), (t, l)
    assert more > 0 or len(failed) >= 10


@pytest.mark.parametrize("sides", [[1, 1, 3], [3], [5], [7], [1, 3, 5, 7]], ids=["p1", "p3", "p5", "p7", "mixed"])
@pytest.mark.parametrize("feed", [0, 2], ids=["shares", "fed"])
def test_beside_a_large_layer(sides, feed):
    """Small layers of every side whose v replaces the residual because of a large layer in the plan (one without anything to keep, so that the
    oracle has little to do): with the tiles in fixed shares and from the work feed, which does not decide the form."""
    from paper_2312_17530_amd.session import Session
    shapes = [(40, 40), (33, 512), (16, 256), (17, 257), (48, 768), (18, 259), (35, 1030), (15, 511), (64, 27), (1, 700), (3, 2100),
              (130, 131), (49, 1028), (32, 513), (50, 64), (34, 300), (64, 520), (4096, 8200)]
    ratios = [0.9, 0.02, 0.02, 0.05, 0.03, 0.05, 0.02, 0.05, 0.03, 0.02, 0.02, 0.04, 0.01, 0.05, 0.0, 0.02, 0.02, 0.0]
    frozen, tied, hot, big = {13}, {15}, 16, 17
    ps = [sides[l % len(sides)] for l in range(big)] + [3]
    rng = np.random.default_rng(170 + sides[0] + len(sides))
    s = Session(shapes, 3, 0.5, ratios, ps, in_place=True, work_feed=feed)
    assert s.plan.replaces_residual
    small = Session(shapes[:big], 3, 0.5, ratios[:big], [3] * big, in_place=True, work_feed=feed)
    assert not small.plan.replaces_residual
    paths = []
    for t in range(5):
        scale = 10.0 if t == 4 else 1e-2
        grads = [np.zeros(sh, np.float32) if l in frozen else (rng.integers(-1, 2, sh) * scale).astype(np.float32) if l in tied else
                 (rng.standard_normal(sh, np.float32) * np.float32(scale)) for l, sh in enumerate(shapes)]
        grads[hot][16:32, :256] *= np.float32(30.0)
        resid = s.unpack(s.residual)
        s.set_grad(grads)
        s.compress()
        paths.append(binding.rsdgc_last_paths(s.plan, s.workspace))
        if t in (1, 2):
            continue
        after = s.unpack(s.residual)
        for l, (idx, val, centres, _) in enumerate(s.results()):
            if l == big:
                assert len(idx) == 0 and np.array_equal(_bits(after[l]), _bits(resid[l] + grads[l])), t
                continue
            o = oracle.compress_layer(grads[l], resid[l], ps[l], 0.5, ratios[l])
            assert np.array_equal(idx, o.idx) and np.array_equal(centres, o.centres), (t, l)
            assert np.array_equal(_bits(val), _bits(o.val)) and np.array_equal(_bits(after[l]), _bits(o.r_new)), (t, l)
    assert paths[0].count(0) >= 10 and paths[4].count(1) > paths[3].count(1), paths
