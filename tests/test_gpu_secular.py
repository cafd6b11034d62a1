"""The sweeps' sign function (the dispersion function in minors) against the
oracle's determinant: layer counts around the rescaling periods (4 layers in
FP32, 8 in FP64), wavelengths whose layers take every branch of the potential
terms, and grids below and above the half-space's S velocity.  The bar is the
parity bar: exact index outside the FP64 noise band, roots within 1e-6."""
import math

import numpy as np
import pytest

import paper_2003_02256_amd as M
import workloads as WL
from test_gpu_parity import compare, dev_batch, dev_curve, oracle_curve

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev(gpu):
    import torch
    return torch, torch.device("cuda:0")


@pytest.fixture(scope="module")
def ctx(gpu):
    c = M.Context(0, 1 << 30)
    yield c
    c.close()


def profile(n, h=None):
    rng = np.random.Generator(np.random.PCG64(900 + n))
    m = WL.increasing_profile(rng, n)
    if n > 3:  # one slower layer
        WL.apply_inversion(rng, m, 1.0)
    if h is not None:
        m = WL.Model(np.full(n, h), m.alpha, m.beta, m.rho)
    return m


@pytest.mark.parametrize("prec", [M.MASW_PREC_FP64, M.MASW_PREC_SPLIT])
@pytest.mark.parametrize("n", [0, 1, 3, 4, 5, 7, 8, 9, 17])
def test_layer_counts(torch_dev, ctx, n, prec):
    m = profile(n)
    lam = np.array([0.8, 4.0, 15.0, 60.0])
    c = WL.uniform_grid(60.0, 1.0, 600)
    want = oracle_curve(lam, c, m)
    compare(f"N={n} prec={prec}", dev_curve(torch_dev, ctx, c, lam, m, prec), *want, lam, c, m)
    got = dev_batch(torch_dev, ctx, c, [m, m], [lam, lam], prec)  # staged records
    for half in (slice(0, 4), slice(4, 8)):
        compare(f"batch N={n} prec={prec}", [g[half] for g in got], *want, lam, c, m)


@pytest.mark.parametrize("prec", [M.MASW_PREC_FP64, M.MASW_PREC_SPLIT])
@pytest.mark.parametrize("above", [False, True])
@pytest.mark.parametrize("kh", [0.05, 1.9, 2.1, 6.0, 40.0])
def test_potential_branches(torch_dev, ctx, kh, above, prec):
    # k h sqrt|x| on both sides of 2, and cos/sin of large arguments (c up to
    # 5 beta of the half-space)
    m = profile(6, h=2.0)
    lam = np.array([2.0 * math.pi * 2.0 / kh])
    b = float(m.beta[-1])
    c = WL.uniform_grid(1.01 * b, 0.005 * b, 800) if above else WL.uniform_grid(0.2 * b, 0.002 * b, 380)
    got = dev_curve(torch_dev, ctx, c, lam, m, prec)
    want = oracle_curve(lam, c, m)
    if above:  # (at k h = 40 the picked step holds three roots; the oracle's bisection ends at another one)
        assert list(got[1]) == want[0] and list(got[2]) == want[1]
    else:
        compare(f"kh={kh} prec={prec}", got, *want, lam, c, m)


@pytest.mark.parametrize("ulps", [1, 8, 64])
def test_a_pick_is_a_change_of_the_determinant(torch_dev, ctx, ulps):
    # a grid of neighbouring doubles across a root: the sweep's sign and the
    # determinant's round differently there, and the reported step has to be a
    # change of the latter (the sign map's)
    m = profile(9)
    lam0 = np.array([12.0])
    root = float(dev_curve(torch_dev, ctx, WL.uniform_grid(60.0, 1.0, 600), lam0, m, M.MASW_PREC_FP64)[3][0])
    step = np.spacing(root) * ulps
    for lam in lam0 * (1.0 + np.arange(-8, 9) * 2e-16 * ulps):
        c = root + (np.arange(2001) - 1000) * step
        ct, idx, st, _ = dev_curve(torch_dev, ctx, c, np.array([lam]), m, M.MASW_PREC_FP64)
        sig, _ = ctx.sign_map(c, np.array([lam]), m, M.MASW_PREC_FP64)
        s = sig[0]
        if idx[0] < 0:
            assert np.all(s == s[0])
            continue
        assert s[idx[0]] != s[idx[0] - 1] and ct[0] == c[idx[0]]


@pytest.mark.parametrize("flags", [0, M.MASW_NO_REFINE])
@pytest.mark.parametrize("prec", [M.MASW_PREC_FP64, M.MASW_PREC_SPLIT])
@pytest.mark.parametrize("extra", [1, 700])
def test_sweep_and_picks_in_launches_of_their_own(torch_dev, ctx, extra, prec, flags):
    # just above the item count (48 per SIMD) from which the sweep, the picks
    # and the picks that eight lanes do not settle are separate launches:
    # outputs equal those of the same items in batches below it, bit for bit.
    # The models have poles, changes below the grid, no change at all and
    # modes in the grid's last steps; some are invalid.
    torch, dev = torch_dev
    n = 48 * 4 * torch.cuda.get_device_properties(dev).multi_processor_count + extra
    rng = np.random.Generator(np.random.PCG64(77 + extra))
    models, lambdas, left = [], [], n
    while left > 0:
        i = len(models)
        m = WL.random_model(rng, int(rng.integers(1, 20))) if i % 3 == 0 else profile(int(rng.integers(0, 12)))
        if i % 50 == 7:
            m = WL.Model(m.h, m.alpha, -m.beta, m.rho)
        w = min(left, int(rng.integers(1, 400)))
        lambdas.append(np.sort(np.exp(rng.uniform(np.log(0.5), np.log(200.0), size=w))))
        if i % 20 == 3:
            lambdas[-1][w // 2] = np.inf
        models.append(m)
        left -= w
    c = WL.uniform_grid(120.0, 0.7, 1100)
    got = dev_batch(torch_dev, ctx, c, models, lambdas, prec, flags)
    assert len(got[1]) == n
    h = len(models) // 2
    parts = [dev_batch(torch_dev, ctx, c, models[s], lambdas[s], prec, flags) for s in (slice(0, h), slice(h, None))]
    for x, *y, what in zip(got, *parts, ("C_t", "idx", "status", "c_ref")):
        np.testing.assert_array_equal(x, np.concatenate(y), err_msg=what)
    if flags == 0:
        compare("staged picks", [g[:20] for g in got], *oracle_curve(lambdas[0][:20], c, models[0]), lambdas[0][:20],
                c, models[0])
