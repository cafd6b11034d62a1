"""Batches of mostly empty models: more models than wavelengths, in each form of
the inertia search's launch (64, 32 and 8 lanes a wavelength, and the
persistent grid), against the walk."""
import numpy as np
import pytest

import paper_2003_02256_amd as M
import workloads as WL
from test_gpu_parity import dev_batch

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


@pytest.mark.parametrize("n_models", [2, 8000, 20011])
@pytest.mark.parametrize("n", [7, 2049, 4096, 4097, 33000])
def test_more_models_than_wavelengths(torch_dev, ctx, n, n_models):
    rng = np.random.Generator(np.random.PCG64(n + n_models))
    kinds = [WL.two_layer_model(), WL.increasing_profile(rng, 5), WL.random_model(rng, 3),
             WL.Model(np.zeros(0), np.array([700.0]), np.array([400.0]), np.array([2000.0]))]
    owners = np.sort(rng.choice(n_models, size=min(n_models, max(2, n // 9)), replace=False))
    counts = np.zeros(n_models, int)
    np.add.at(counts, owners[rng.integers(0, len(owners), n)], 1)
    models = [kinds[i % 4] for i in range(n_models)]
    lambdas = [np.sort(rng.uniform(1.0, 60.0, k)) for k in counts]
    c = WL.uniform_grid(60.0, 0.5, 901)
    walk = dev_batch(torch_dev, ctx, c, models, lambdas, M.MASW_PREC_FP64)
    got = dev_batch(torch_dev, ctx, c, models, lambdas, M.MASW_PREC_FP64, M.MASW_SEARCH_INERTIA)
    st = ctx.stats()
    for x, y, what in zip(walk, got, ("C_t", "idx", "status", "c_ref")):
        np.testing.assert_array_equal(y, x, err_msg=what)
    assert st["useful_evals"] == int(np.sum(np.where(walk[1] >= 0, walk[1] + 1, len(c))))
    assert st["inertia_evals"] >= n
