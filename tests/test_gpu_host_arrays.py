"""Host-array calls pass their inputs and outputs through one pinned block
each way while they fit (256 KiB), and copy array by array beyond that: on
both sides of the limits the outputs equal the device-array call's bit for
bit, call after call with other inputs, and with several threads at once."""
import threading

import numpy as np
import pytest

import paper_2003_02256_amd as M
import workloads as WL
from test_gpu_parity import dev_batch, dev_curve

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev(gpu):
    import torch
    return torch, torch.device("cuda:0")


def same(a, b):
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("w", [1, 30, 10900, 11000])  # outputs of 24 bytes a wavelength: limit near 10,922
@pytest.mark.parametrize("n_c", [2, 900, 32600, 32800])  # grid of 8 bytes a point: limit near 32,700
def test_curves_around_the_limits(torch_dev, gpu, n_c, w):
    m = WL.two_layer_model()
    with M.Context(0, 256 << 20) as ctx:
        for shift in (0.0, 3.0):
            c = np.linspace(150.0 + shift, 390.0, n_c)
            lam = np.linspace(2.0 + shift, 60.0, w)
            same(ctx.curve(c, lam, m, M.MASW_PREC_FP64), dev_curve(torch_dev, ctx, c, lam, m, M.MASW_PREC_FP64))


def test_batches_and_threads(torch_dev, gpu):
    rng = np.random.Generator(np.random.PCG64(31))
    models = [WL.increasing_profile(rng, int(n)) for n in rng.integers(1, 12, 9)]
    lambdas = [np.linspace(2.0, 30.0, int(n)) for n in rng.integers(1, 40, 9)]
    c = WL.uniform_grid(60.0, 0.5, 1200)
    with M.Context(0, 256 << 20) as ctx:
        want = dev_batch(torch_dev, ctx, c, models, lambdas, M.MASW_PREC_FP64)
        same(ctx.batch(c, models, lambdas, prec=M.MASW_PREC_FP64), want)
        off = np.concatenate([[0], np.cumsum([len(l) for l in lambdas])])
        bad = []

        def run(i):
            for _ in range(10):
                got = ctx.curve(c, lambdas[i], models[i], M.MASW_PREC_FP64)
                if any(not np.array_equal(x, y[off[i]:off[i + 1]], equal_nan=True) for x, y in zip(got, want)):
                    bad.append(i)

        threads = [threading.Thread(target=run, args=(i,)) for i in range(6)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not bad
