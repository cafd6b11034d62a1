"""A grid step with three roots, the first two between two neighbours of the
eight points that are evaluated first: the refined root is the first one that
64 equally spaced points show (two slow layers apart have their modes in
pairs)."""
import numpy as np
import pytest

import oracle as O
import paper_2003_02256_amd as M
import workloads as WL

pytestmark = pytest.mark.gpu
PR = O.propagator


@pytest.fixture(scope="module")
def ctx(gpu):
    c = M.Context(0, 256 << 20)
    yield c
    c.close()


def pair_model(h, sep, b3=100.4):
    """Two slow layers h apart by sep, and a third further down."""
    be = np.array([300.0, 100.0, 300.0, 100.0, 300.0, b3, 600.0])
    return WL.Model(np.array([3.0, h, sep, h, 12.0, h]), 2.0 * be, be,
                    np.array([2000.0, 1800.0, 2000.0, 1800.0, 2000.0, 1800.0, 2100.0]))


# (model, wavelength, step, its three roots); no layer denominator is negative
# and there is no root below
CASES = [(pair_model(2.0, 2.0), 3.0, (142.1, 144.7), (142.208, 142.388, 144.632)),
         (pair_model(2.0, 2.0, 100.8), 3.0, (142.15, 145.3), (142.208, 142.388, 145.180)),
         (pair_model(1.5, 3.0), 3.0, (171.4, 176.4), (171.604, 171.756, 176.264)),
         (pair_model(2.0, 4.0), 4.0, (171.4, 176.4), (171.576, 171.736, 176.264))]


@pytest.mark.parametrize("m,lam,step,roots", CASES)
def test_classified_root_is_the_first(ctx, m, lam, step, roots):
    # the oracle's root, by bisection between the first root's neighbourhood
    alone = np.array([roots[0] - 0.1, roots[0] + 0.1])
    want_cls, want = PR.classify(lam, alone, 1, m)
    assert want_cls == PR.PICK_MODE
    k = 2.0 * np.pi / lam
    sg = [np.sign(PR.secular(k, c, m)) for c in np.linspace(*step, 64)]
    assert int(np.sum(np.diff(sg) != 0)) == 3 and int(np.sum(np.diff(sg[::9]) != 0)) == 1
    c = np.array([step[0], step[1], step[1] + 10.0])
    for copies in (1, 9):
        cls, sec = ctx.classify(c, [m], [np.full(copies, lam)], np.ones(copies, np.int32))
        assert np.all(cls == M.MASW_PICK_MODE)
        assert np.all(np.abs(sec - want) <= 1e-9 * want), (sec, want)


# Every form of the sweep and of the inertia search: alone (a fused launch), in
# staged launches of 5000 and of 49,153 wavelengths and more (the sweep and the
# picks apart), and 64, 32 and 8 lanes a wavelength.
@pytest.mark.parametrize("search", ["walk", "split", "inertia"])
@pytest.mark.parametrize("copies", [1, 2100, 5000, 33000, 60000])
def test_refined_root_is_the_first(ctx, search, copies):
    prec = M.MASW_PREC_SPLIT if search == "split" else M.MASW_PREC_FP64
    flags = M.MASW_SEARCH_INERTIA if search == "inertia" else 0
    for m, lam, step, roots in CASES:
        alone = np.array([roots[0] - 0.1, roots[0] + 0.1])
        want = PR.classify(lam, alone, 1, m)[1]
        n = 1100 if search == "split" else 30      # a split call on fewer points is the FP64 walk
        c = np.r_[np.linspace(120.0, step[0], n), step[1], step[1] + 1.0 + np.arange(5.0)]
        if copies == 1:
            ct, idx, st, ref = ctx.curve(c, np.array([lam]), m, prec, flags)
        else:
            ct, idx, st, ref = ctx.batch(c, [m], [np.full(copies, lam)], prec, flags)
        assert np.all(idx == n) and np.all(ct == step[1]) and np.all(st == M.MASW_STATUS_FOUND)
        assert np.all(np.abs(ref - want) <= 2e-9 * want), (ref[:3], want)
