"""A batched step whose new scores take the old ones' place (phi is phi_prev),
and whose particles take the previous ones': every step kernel reads its inputs
before it writes, so the results are those of separate arrays, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2312_08684_amd import smsq
from test_gpu_parity import DEV, _svgd_case, announce, dev, tdt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("n,step_kernel", [(20, "auto"), (64, "auto"), (20, "wave"), (64, "valu"), (96, "auto"),
                                           (600, "auto")])
def test_scores_and_particles_in_place(n, step_kernel, dt):
    announce("in place", n, step_kernel, dt)
    B = 3
    wl, desc, xp, x, z, mask = _svgd_case("range2d", n, n, 60, dt)
    td, model = tdt(dt), smsq.Model(desc)
    rep = lambda a, t: dev(np.repeat(a[None], B, 0), t)
    z, mask = rep(z, td), None if mask is None else rep(mask, torch.uint8)
    scores = dev(np.random.default_rng(6).normal(size=(B, n)), td)
    res = []
    for same in (False, True):
        xg, phi_prev = rep(xp, td), scores.clone()
        x_prev = xg if same else xg.clone()
        phi = phi_prev if same else torch.empty_like(phi_prev)
        psi = torch.empty((B, n), dtype=torch.int32, device=DEV)
        ws = smsq.workspace()
        smsq.batch_step(model, dt, 2, x_prev, phi_prev, z, mask, xg, smsq.opts(3, 0.005, step_kernel=step_kernel),
                        seed=12, phi=phi, psi=psi, ws=ws)
        assert smsq.device_status(ws) == smsq.OK
        res.append((xg, phi, psi))
    for a, b in zip(*res):
        assert torch.equal(a, b)
