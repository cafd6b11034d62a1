"""masw_classify_picks with idx and pick_class in one array: the classes replace
the indices, also those of picks that a second launch finishes."""
import numpy as np
import pytest

import paper_2003_02256_amd as M
import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c", [np.array([100.0, 222.0, 300.0]),      # 122 m/s wide: all deferred
                               WL.uniform_grid(50.0, 0.1, 9501)])
def test_classes_replace_the_indices(gpu, c):
    import torch
    dev = torch.device("cuda:0")
    models = [WL.two_layer_model(), WL.increasing_profile(np.random.Generator(np.random.PCG64(3)), 6)]
    lambdas = [WL.log_spaced(4.0, 10.9, 40), WL.log_spaced(3.0, 30.0, 25)]
    arrs = [torch.as_tensor(a, device=dev) for a in M.flatten_models(models, lambdas)]
    with M.Context(0, 256 << 20) as ctx:
        idx = np.ones(65, np.int32) if len(c) == 3 else ctx.batch(c, models, lambdas, prec=M.MASW_PREC_FP64)[1]
        idx[7] = 0                                                    # one without a bracket
        want, want_sec = ctx.classify(c, models, lambdas, idx)
        both = torch.as_tensor(idx, device=dev)
        sec = torch.empty(65, dtype=torch.float64, device=dev)
        M.masw_classify_picks(ctx.ctx, torch.as_tensor(c, device=dev), *arrs, both, 0, None, both, sec)
        torch.cuda.synchronize()
        assert np.array_equal(both.cpu().numpy(), want)
        np.testing.assert_array_equal(sec.cpu().numpy(), want_sec)
        assert want[7] == M.MASW_PICK_NONE and np.sum(want == M.MASW_PICK_MODE) > 8
