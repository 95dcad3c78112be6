"""Small sets in FP32 over many iterations: the error of their particles against
the oracle, over their displacement, is no larger than that of the kernels that
took such sets before (matrix-core step above 32 particles)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2312_08684_amd import scenarios as S
from paper_2312_08684_amd import smsq
from test_gpu_parity import DEV, announce, dev, host

pytestmark = pytest.mark.gpu


# the rms error of the earlier kernels on these 40 sets, and a seventh for the choice of sets
@pytest.mark.parametrize("name,n,L,step,bound", [("range2d", 48, 100, 0.005, 1.84e-06),
                                                 ("range2d", 64, 100, 0.005, 1.91e-06),
                                                 ("cv4d", 40, 50, 0.005, 5.79e-06),
                                                 ("cv4d", 48, 50, 0.005, 5.87e-06),
                                                 ("cv4d", 64, 50, 0.005, 6.45e-06),
                                                 ("arm7", 40, 50, 1e-05, 8.95e-07),
                                                 ("arm7", 48, 50, 1e-05, 9.39e-07),
                                                 ("growth1d", 48, 100, 0.05, 1.25e-06),
                                                 ("growth1d", 64, 100, 0.05, 1.30e-06)])
def test_error_after_many_iterations(name, n, L, step, bound):
    announce("small sets accuracy", name, n, L)
    errs = []
    for seed in range(40):
        wl = S.make_workload(name, B=1, seed=seed + 100, T=3)
        desc, rng = wl.model, np.random.default_rng(seed)
        f32 = lambda a: a.astype(np.float32).astype(np.float64)
        sd = np.sqrt(desc.q_var[:desc.d])
        xp = wl.truth[0, 1][None] + 2 * sd * rng.normal(size=(n, desc.d))
        mu = np.stack([O.transition_mean(desc, 2, v) for v in xp])
        x = f32(mu[rng.integers(n, size=n)] + sd * rng.normal(size=(n, desc.d)))
        xp, z, mask = f32(xp), f32(wl.z[0, 1]), None if wl.mask is None else wl.mask[0, 1]
        eps = float(np.float32(step))
        xo, _, _ = O.svgd_step(desc, 2, xp, None, z, mask, x, L, eps)
        xg, td = dev(x, torch.float32), torch.float32
        smsq.svgd_step(smsq.Model(desc), "f32", 2, dev(xp, td), None, dev(z, td),
                       None if mask is None else dev(mask, torch.uint8), xg, smsq.opts(L, eps), ws=smsq.workspace())
        errs.append(np.linalg.norm(host(xg) - xo) / np.linalg.norm(xo - x))
    rms = float(np.sqrt(np.mean(np.square(errs))))
    print("rms error over the displacement %.2e" % rms)
    assert rms <= bound
