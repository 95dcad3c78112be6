"""Matrix-core step where its 16-bit operand pieces are short of range or bits:
tight clouds far from their transition means, one particle far from all others,
bandwidths far below the spread.

One iteration against the oracle's scores and Stein direction at the bandwidth
the step reports (the median of rounded distances is another matter).  The
kernel values of such sets come from FP32 differences of particles held
relative to the transition means: for a cloud a fraction f of its offset wide,
an exponent beta |dx|^2 of up to 20 is off by 20 * 4 * 2^-24 / f, 1e-2 at the
narrowest (f = 5e-4), hence 2e-2 of the displacement, with four roundings of the
positions."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2312_08684_amd import smsq
from test_gpu_parity import DEV, _svgd_case, announce, dev, host

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24


def one_iteration(desc, xp, z, mask, x, step, bw_scale=1.0, log_w=None, iters=1):
    """Particles after an iteration on the matrix cores and their bandwidth."""
    td = torch.float32
    xg, hg, ws = dev(x, td), torch.zeros(iters, dtype=td, device=DEV), smsq.workspace()
    smsq.svgd_step(smsq.Model(desc), "f32", 2, dev(xp, td), None if log_w is None else dev(log_w, td), dev(z, td),
                   None if mask is None else dev(mask, torch.uint8), xg,
                   smsq.opts(iters, step, bw_scale, step_kernel="mfma"), h_out=hg, ws=ws)
    assert smsq.device_status(ws) == smsq.OK
    return host(xg).astype(np.float64), float(host(hg)[0])


def expected(desc, xp, z, mask, x, step, h, log_w=None):
    s = O.scores(desc, 2, xp, log_w, z, mask, x)
    return x + step * O.stein_phi(x, s, h)


def f32(a):
    return a.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("name", ["growth1d", "range2d", "cv4d", "arm7"])
@pytest.mark.parametrize("n", [60, 100, 600])
@pytest.mark.parametrize("kind", ["tight", "outlier", "small_bandwidth"])
def test_far_beyond_the_spread(kind, n, name):
    announce("matrix step range", kind, n, name)
    wl, desc, xp, x, z, mask = _svgd_case(name, n, 90, 70, "f32")
    sd, mean = x.std(0), x.mean(0)
    bw_scale, step = 1.0, 0.005
    if kind == "small_bandwidth":
        bw_scale, step = 1e-7, 0.005 * n * float(sd.max()) / (1 + np.abs(O.scores(desc, 2, xp, None, z, mask, x)).max())
    else:
        width = 5e-4 if kind == "tight" else 1e-2
        # the cloud moves to five deviations of its place along every axis
        x = mean + 5.0 * sd * (1.0 if kind == "tight" else 0.0) + 5.0 * width * (x - mean)
        if kind == "outlier":
            x[n // 3] = mean + 1e4 * 5.0 * width * sd
        x = f32(x)
        step = float((width * sd).min()) ** 2
    xg, h = one_iteration(desc, xp, z, mask, x, step, bw_scale)
    xo = expected(desc, xp, z, mask, x, step, h)
    rest = np.arange(n) != n // 3 if kind == "outlier" else np.arange(n) >= 0
    err, disp = np.linalg.norm((xg - xo)[rest]), np.linalg.norm((xo - x)[rest])
    print("h %.3e, error %.3e of the displacement %.3e" % (h, err / disp, disp))
    assert np.isfinite(xg).all()
    assert err <= 2e-2 * disp + 4 * EPS * np.linalg.norm(x[rest])


@pytest.mark.parametrize("name", ["growth1d", "range2d", "cv4d", "arm7"])
@pytest.mark.parametrize("n", [70, 600])
def test_equal_particles_stay_finite(n, name):
    """Distances of equal particles are roundings, and their median a bandwidth
    of that size: kappa is one all the same, and the particles move alike."""
    announce("matrix step equal", n, name)
    wl, desc, xp, x, z, mask = _svgd_case(name, n, 90, 71, "f32")
    for i in range(8):
        xe = np.repeat(x[i:i + 1], n, 0)
        xg, h = one_iteration(desc, xp, z, mask, xe, 1e-6, iters=5)
        assert np.isfinite(xg).all() and np.abs(xg - xg[0]).max() == 0


@pytest.mark.parametrize("n", [512, 1024])
def test_small_bandwidth_on_several_workgroups(n):
    announce("matrix step small bandwidth, several workgroups", n)
    from paper_2312_08684_amd import scenarios as S
    wl = S.make_workload("cv4d", B=1, seed=9, T=2, n=n, n_iter=3)
    model, td = smsq.Model(wl.model), torch.float32
    x0, z = dev(wl.x0[:1], td), dev(wl.z[:1, :2], td)
    mk = None if wl.mask is None else dev(wl.mask[:1, :2], torch.uint8)
    res = []
    for sk in ("coop", "valu"):
        parts = torch.zeros((1, 2, n, 4), dtype=td, device=DEV)
        ws = smsq.workspace(model.workspace_size("f32", 1, 2, n))
        smsq.run_batch(model, "f32", x0, z, mk, n, smsq.opts(3, 0.05, 1e-7, step_kernel=sk), 5, particles=parts, ws=ws)
        assert smsq.device_status(ws) == smsq.OK
        res.append(host(parts).astype(np.float64)[0, 0])
    # FP32 sums in another order, three iterations of a step of 0.05 / n scores
    assert np.linalg.norm(res[0] - res[1]) <= 1e-5 * np.linalg.norm(res[1])
