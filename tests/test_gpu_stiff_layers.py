"""Walks over velocities far below a layer's S velocity, where the sweeps' sign
function in minors is rounding noise and the elimination is not: a thin stiff
layer over a soft half-space.  The pick is the first change of sign(det K)
along the grid, as the sign map (the elimination at every grid point) has it,
and lies where 33 digits put it (PICKS, on a grid of 1 m/s)."""
import math

import numpy as np
import pytest

import paper_2003_02256_amd as M
import workloads as WL
from test_gpu_parity import dev_batch, dev_curve
from test_gpu_serving import submit, wait

pytestmark = pytest.mark.gpu

SLAB = WL.Model(np.array([0.2]), 1.9 * np.array([2300.0, 200.0]), np.array([2300.0, 200.0]), np.array([2000.0] * 2))
PICKS = {60.0: 200.0, 150.0: 198.0, 300.0: 195.0, 450.0: 194.0}
# on velocities above 1/64 of its largest beta, where the sweep is in minors
PLATE = WL.Model(np.array([0.0021]), np.array([8600.0, 2400.0]), np.array([4600.0, 84.0]), np.array([2450.0, 1500.0]))


@pytest.fixture(scope="module")
def torch_dev(gpu):
    import torch
    return torch, torch.device("cuda:0")


@pytest.fixture(scope="module")
def ctx(gpu):
    c = M.Context(0, 1 << 30)
    yield c
    c.close()


def first_changes(ctx, c, lam, m):
    sig, _ = ctx.sign_map(c, lam, m, M.MASW_PREC_FP64)
    return [int(np.argmax(s[1:] != s[:-1])) + 1 if np.any(s[1:] != s[:-1]) else -1 for s in sig]


def check(out, c, lam, want, near=None):
    ct, idx, st, cr = out
    assert list(idx) == want
    for w, i in enumerate(want):
        assert st[w] == M.MASW_STATUS_FOUND and ct[w] == c[i] and c[i - 1] <= cr[w] <= c[i]
        if near is not None:
            assert near[w] - 1.0 < ct[w] <= near[w] + (c[1] - c[0])


# a fused launch; a staged one of a few rounds; shared sweeps of many rounds
@pytest.mark.parametrize("step,n", [(1.0, 420), (0.25, 1680), (0.1, 4200)])
@pytest.mark.parametrize("c0", [1.0, 2.0, 5.0, 10.0])
@pytest.mark.parametrize("prec", [M.MASW_PREC_FP64, M.MASW_PREC_SPLIT])
def test_curve_from_low_velocities(torch_dev, ctx, prec, c0, step, n):
    lam = np.array(list(PICKS))
    c = c0 + step * np.arange(n)
    want = first_changes(ctx, c, lam, SLAB)
    check(dev_curve(torch_dev, ctx, c, lam, SLAB, prec), c, lam, want, list(PICKS.values()))
    two = dev_batch(torch_dev, ctx, c, [SLAB, SLAB], [lam, lam], prec)
    for half in (slice(0, 4), slice(4, 8)):
        check([x[half] for x in two], c, lam, want, list(PICKS.values()))


def test_a_thinner_layer(torch_dev, ctx):
    m = WL.Model(np.array([0.134]), 1.9 * np.array([3306.0, 211.0]), np.array([3306.0, 211.0]), np.array([2000.0] * 2))
    lam, c = np.array([372.0]), 10.0 + 0.1 * np.arange(2500)
    check(dev_curve(torch_dev, ctx, c, lam, m, M.MASW_PREC_FP64), c, lam, [1958], [206.0])


# noise that the rule on velocities does not keep away: the walk is made again
@pytest.mark.parametrize("n_lam", [3, 400, 5000])
def test_a_change_that_the_elimination_does_not_confirm(torch_dev, ctx, n_lam):
    lam = np.linspace(2000.0, 3000.0, n_lam)
    for c in (72.0 + 0.1 * np.arange(119), 72.0 + 0.004 * np.arange(2900)):
        want = first_changes(ctx, c, lam[[0, -1]], PLATE)
        assert min(want) > 0 and all(80.0 < c[i] < 81.0 for i in want)
        ct, idx, st, _ = dev_curve(torch_dev, ctx, c, lam, PLATE, M.MASW_PREC_FP64)
        assert [idx[0], idx[-1]] == want
        assert np.all(st == M.MASW_STATUS_FOUND) and np.all((ct > 80.0) & (ct < 81.0))


# batches on both sides of the line (48 wavelengths per SIMD) above which the
# sweep and the picks are launches of their own
@pytest.mark.parametrize("c0,model,lo,hi", [(1.0, SLAB, 60.0, 450.0), (5.0, SLAB, 60.0, 450.0),
                                            (72.0, PLATE, 2000.0, 3000.0)])
@pytest.mark.parametrize("extra", [-1, 1])
def test_batches_on_both_sides_of_the_staged_line(torch_dev, ctx, extra, c0, model, lo, hi):
    torch, dev = torch_dev
    n = 48 * 4 * torch.cuda.get_device_properties(dev).multi_processor_count + extra
    c = c0 + 0.5 * np.arange(400) if model is SLAB else c0 + 0.01 * np.arange(1190)
    other = WL.two_layer_case().models[0]  # swept in minors
    lams = [np.linspace(lo, hi, n // 2), np.linspace(1.0, 40.0, n - n // 2)]
    got = dev_batch(torch_dev, ctx, c, [model, other], lams, M.MASW_PREC_FP64)
    parts = [dev_curve(torch_dev, ctx, c, l, m, M.MASW_PREC_FP64) for m, l in zip((model, other), lams)]
    for x, *y, what in zip(got, *parts, ("C_t", "idx", "status", "c_ref")):
        np.testing.assert_array_equal(x, np.concatenate(y), err_msg=what)
    some = np.linspace(0, n // 2 - 1, 16).astype(int)
    check([x[some] for x in got], c, lams[0][some], first_changes(ctx, c, lams[0][some], model))


@pytest.mark.parametrize("rounds", [1, 64])
@pytest.mark.parametrize("prec", [M.MASW_PREC_FP64, M.MASW_PREC_SPLIT])
def test_served_requests(ctx, prec, rounds):
    lam = np.array(list(PICKS))
    reqs = [(SLAB, c0 + 0.25 * np.arange(1680), lam) for c0 in (1.0, 5.0)]
    reqs.append((PLATE, 72.0 + 0.004 * np.arange(2900), np.array([2000.0, 2500.0, 3000.0])))
    M.masw_server_start(ctx.ctx, rounds_per_tick=rounds)
    got = [wait(ctx, submit(ctx, c, l, m, prec), len(l))[0] for m, c, l in reqs]
    M.masw_server_stop(ctx.ctx)
    for out, (m, c, l) in zip(got, reqs):
        check(out, c, l, first_changes(ctx, c, l, m))
