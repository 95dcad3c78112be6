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


@pytest.mark.parametrize("n", [100, 600])
def test_one_score_far_beyond_the_others(n):
    """One particle of the growth model at 15,000: its score is 2^30 of the
    others'.  They move as without it, to FP32 rounding (1e-4 is far above it,
    and far below what pieces scaled to the largest value would lose, 2^-10)."""
    announce("matrix step score outlier", n)
    wl, desc, xp, x, z, mask = _svgd_case("growth1d", n, 90, 72, "f32")
    x[n // 2] = 15000.0
    rest = np.arange(n) != n // 2
    s = O.scores(desc, 2, xp, None, z, mask, x)
    assert abs(s[n // 2, 0]) > 2.0 ** 26 * np.abs(s[rest]).max()
    bw_scale = 200.0
    step = float(x[rest].std() / np.abs(O.stein_phi(x, s, O.bandwidth(x, bw_scale)[0])[rest]).max())
    xg, h = one_iteration(desc, xp, z, mask, x, step, bw_scale)
    assert 2.0 / h * 0.5 * np.log2(np.e) * 15000.0 ** 2 < 2.0 ** 20   # (products, not differences)
    xo = expected(desc, xp, z, mask, x, step, h)
    err, disp = np.linalg.norm((xg - xo)[rest]), np.linalg.norm((xo - x)[rest])
    print("h %.3e, error %.3e of the displacement" % (h, err / disp))
    assert err <= 1e-4 * disp + 4 * EPS * np.linalg.norm(x[rest])


@pytest.mark.parametrize("n", [100, 600])
def test_dimensions_of_unequal_scale(n):
    """A linear-Gaussian state whose deviations are 1, 2^-16 and 2^-32, so that
    its scores are 1, 2^16 and 2^32: each dimension moves to FP32 rounding of
    its own displacement."""
    announce("matrix step unequal dimensions", n)
    from paper_2312_08684_amd import scenarios as S
    sd = np.array([1.0, 2.0 ** -16, 2.0 ** -32])
    desc = S.lingauss_model(np.eye(3), np.array([[1.0, 0.0, 0.0]]), sd ** 2, [0.5])  # observes the first one
    rng = np.random.default_rng(7)
    xp = f32(sd * rng.normal(size=(n, 3)))
    x = f32(xp[rng.integers(n, size=n)] + sd * rng.normal(size=(n, 3)))
    z = f32(np.array([0.3]))
    s = O.scores(desc, 2, xp, None, z, None, x)
    step = float(0.3 / np.abs(O.stein_phi(x, s, O.bandwidth(x)[0])[:, 0]).max())
    xg, h = one_iteration(desc, xp, z, None, x, step)
    xo = expected(desc, xp, z, None, x, step, h)
    for c in range(3):
        err, disp = np.linalg.norm((xg - xo)[:, c]), np.linalg.norm((xo - x)[:, c])
        print("dimension %d: error %.3e of the displacement" % (c, err / disp))
        assert err <= 1e-4 * disp


# the rms error of the direction with FP32 matrix products in place of the
# operand pieces, on these inputs: 2.7, 2.9; 2.1, 2.2; 3.7, 3.5 (1e-7), and a
# quarter for the choice of six sets
@pytest.mark.parametrize("name,n,bound", [("range2d", 64, 3.4e-7), ("range2d", 512, 3.6e-7), ("cv4d", 64, 2.6e-7),
                                          ("cv4d", 512, 2.8e-7), ("arm7", 64, 4.6e-7), ("arm7", 512, 4.4e-7)])
def test_direction_is_as_accurate_as_fp32_products(name, n, bound):
    announce("matrix step accuracy", name, n)
    from paper_2312_08684_amd import scenarios as S
    errs = []
    for seed in range(6):
        wl = S.make_workload(name, B=1, seed=seed + 100, T=3)
        desc, rng = wl.model, np.random.default_rng(seed)
        sd = np.sqrt(desc.q_var[:desc.d])
        xp = wl.truth[0, 1][None] + 2 * sd * rng.normal(size=(n, desc.d))
        mu = np.stack([O.transition_mean(desc, 2, v) for v in xp])
        x = f32(mu[rng.integers(n, size=n)] + sd * rng.normal(size=(n, desc.d)))
        xp, z, mask = f32(xp), f32(wl.z[0, 1]), None if wl.mask is None else wl.mask[0, 1]
        # a step so large that the positions' own rounding counts for nothing
        phi = O.stein_phi(x, O.scores(desc, 2, xp, None, z, mask, x), O.bandwidth(x)[0])
        step = float(np.float32(1e3 * np.linalg.norm(x) / np.linalg.norm(phi)))
        xg, h = one_iteration(desc, xp, z, mask, x, step)
        xo = expected(desc, xp, z, mask, x, step, h)
        errs.append(np.linalg.norm(xg - xo) / np.linalg.norm(xo - x))
    rms = float(np.sqrt(np.mean(np.square(errs))))
    print("rms error of the direction %.2e" % rms)
    assert rms <= bound
