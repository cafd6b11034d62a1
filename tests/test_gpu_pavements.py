"""The split path on a stiff layer over a much softer one: walked in FP64 where
the grid starts below 1/12 of the stiff layer's velocity (no check of a
candidate is made then), swept in FP32 above; the same picks either way."""
import numpy as np
import pytest

import paper_2003_02256_amd as M
import workloads as WL
from test_gpu_parity import compare, dev_batch, dev_curve, oracle_curve
from test_gpu_serving import submit, wait

pytestmark = pytest.mark.gpu
LAM = np.array([0.7, 2.0, 6.0, 20.0])


@pytest.fixture(scope="module")
def torch_dev(gpu):
    import torch
    return torch, torch.device("cuda:0")


@pytest.fixture(scope="module")
def ctx(gpu):
    c = M.Context(0, 1 << 30)
    yield c
    c.close()


def model(n, stiff, soft):
    """n layers of 0.5 m and 300 m/s over 400 m/s, layer `stiff` of 1200 m/s and
    `soft` (n: the half-space) of 200 m/s."""
    be = np.full(n + 1, 300.0)
    be[-1] = 400.0
    be[stiff], be[soft] = 1200.0, 200.0
    return WL.Model(np.full(n, 0.5), 2.0 * be, be, np.linspace(1800.0, 2200.0, n + 1))


# layer counts around a wavefront's 64 (a fused launch holds up to 64)
@pytest.mark.parametrize("n,stiff,soft", [(1, 0, 1), (3, 0, 2), (63, 0, 62), (63, 62, 63), (64, 63, 64), (64, 0, 63),
                                          (65, 63, 64), (65, 64, 65), (130, 10, 129), (130, 127, 128)])
@pytest.mark.parametrize("c0,fp64", [(99.0, True), (101.0, False)])
def test_where_the_split_path_walks(torch_dev, ctx, n, stiff, soft, c0, fp64):
    m = model(n, stiff, soft)
    c = WL.uniform_grid(c0, 0.25, 1100)
    want = dev_curve(torch_dev, ctx, c, LAM, m, M.MASW_PREC_FP64)
    for models in (1, 3):
        if models == 1:
            got = dev_curve(torch_dev, ctx, c, LAM, m, M.MASW_PREC_SPLIT)
        else:
            got = [x[4:8] for x in dev_batch(torch_dev, ctx, c, [m] * 3, [LAM] * 3, M.MASW_PREC_SPLIT)]
        assert (ctx.stats()["check_evals"] == 0) == fp64
        for x, y, what in zip(got, want, ("C_t", "idx", "status", "c_ref")):
            np.testing.assert_array_equal(x, y, err_msg=what)
    if n <= 3:
        compare(f"N={n}", got, *oracle_curve(LAM, c, m), LAM, c, m)


# the other way round, or half as slow, no FP64 walk
@pytest.mark.parametrize("be", [[200.0, 1200.0, 3000.0], [400.0, 201.0, 600.0]])
def test_where_it_does_not(torch_dev, ctx, be):
    be = np.array(be)
    m = WL.Model(np.array([2.0, 2.0]), 2.0 * be, be, np.full(3, 2000.0))
    c = WL.uniform_grid(30.0, 0.25, 1500)
    want = dev_curve(torch_dev, ctx, c, LAM, m, M.MASW_PREC_FP64)
    got = dev_curve(torch_dev, ctx, c, LAM, m, M.MASW_PREC_SPLIT)
    assert ctx.stats()["check_evals"] > 0
    for x, y in zip(got, want):
        np.testing.assert_array_equal(x, y)


def test_large_batches_and_served_requests(torch_dev, ctx):
    torch, dev = torch_dev
    n = 32 * 4 * torch.cuda.get_device_properties(dev).multi_processor_count + 1
    c = WL.uniform_grid(60.0, 0.3, 1100)
    ms = [model(5, 0, 2), model(5, 4, 5), WL.increasing_profile(np.random.Generator(np.random.PCG64(1)), 6)]
    lams = [np.geomspace(0.7, 30.0, n // 3 + 1)] * 3
    got = dev_batch(torch_dev, ctx, c, ms, lams, M.MASW_PREC_SPLIT)
    want = dev_batch(torch_dev, ctx, c, ms, lams, M.MASW_PREC_FP64)
    for x, y, what in zip(got, want, ("C_t", "idx", "status", "c_ref")):
        np.testing.assert_array_equal(x, y, err_msg=what)
    M.masw_server_start(ctx.ctx)
    served = [wait(ctx, submit(ctx, c, LAM, m, M.MASW_PREC_SPLIT), 4)[0] for m in ms]
    M.masw_server_stop(ctx.ctx)
    for out, m in zip(served, ms):
        for x, y in zip(out, dev_curve(torch_dev, ctx, c, LAM, m, M.MASW_PREC_FP64)):
            np.testing.assert_array_equal(x, y)
