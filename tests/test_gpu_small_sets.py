"""The small-set step kernel (sixteen lanes a particle; the default up to 64
particles) against the oracle and, where it is selected by a rule, against the
workgroup vector-ALU kernel over every form of a batched step.

Particle counts around its waves of four, its sixteen-lane strides, the
register blocks of its selection (256, 512 and 1024 pairs: 23, 32 and 45
particles) and the counts from which the last waves have two duties (57, 61).
Tolerances: those of a teacher-forced step (FP32 1e-4, FP64 1e-10); between the
two kernels, whose sums differ in order only, the same."""
import numpy as np
import pytest
import torch

from paper_2312_08684_amd import smsq
from test_gpu_parity import DEV, TOL_X, _compare_svgd, _svgd_case, announce, dev, host, tdt

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (2, 15), (3, 16), (4, 17), (5, 64), (16, 1), (17, 33), (23, 23), (24, 65), (32, 32), (33, 127),
         (45, 45), (46, 128), (56, 56), (57, 20), (61, 64), (64, 64), (64, 128)]


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("n,n_prev", SIZES)
def test_sizes(n, n_prev, dt):
    announce("small set", n, n_prev, dt)
    name = ("range2d", "cv4d", "growth1d", "lingauss")[(n + n_prev) % 4]
    wl, desc, xp, x, z, mask = _svgd_case(name, n, n_prev, 40 + n, dt)
    _compare_svgd(desc, dt, xp, None, z, mask, x, 12, 0.005)


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("name,n,step", [("arm7", 20, 1e-5), ("arm7", 48, 1e-5), ("arm7", 64, 1e-5),
                                         ("scenario_b", 30, 1e-4), ("scenario_d", 20, 2e-4), ("scenario_d", 40, 2e-4)])
def test_families(name, n, step, dt):
    announce("small set", name, n, dt)
    wl, desc, xp, x, z, mask = _svgd_case(name, n, n, 41, dt)
    _compare_svgd(desc, dt, xp, None, z, mask, x, 20, step)


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("variant", ["weights", "zero_weights", "mean_reading", "per_step_bw", "imq", "matern32",
                                     "ties_2x5", "ties_4x4", "ties_2x10", "ties_8x8", "ties_1x30"])
def test_variants(variant, dt):
    announce("small set", variant, dt)
    n, n_prev, copies = 48, 70, 1
    if variant.startswith("ties_"):
        n, copies = (int(v) for v in variant[5:].split("x"))
    wl, desc, xp, x, z, mask = _svgd_case("range2d", n * copies, n_prev, 42, dt)
    x = np.repeat(x[:n], copies, axis=0)
    log_w, bw_mode, trans_mode, kernel = None, 0, 0, 0
    if "weights" in variant:
        w = np.random.default_rng(3).dirichlet(np.ones(n_prev))
        if variant == "zero_weights":
            w[:10] *= 1e-30   # a first stretch of sources that count nothing
        log_w = np.log(w).astype(np.float32).astype(np.float64)
    if variant == "mean_reading":
        trans_mode = 1
    if variant == "per_step_bw":
        bw_mode = 1
    if variant in ("imq", "matern32"):
        kernel = smsq.KERNELS[variant]
    _compare_svgd(desc, dt, xp, log_w, z, mask, x, 10, 0.005, 1.0, bw_mode, trans_mode, kernel)


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("name,n,n_prev,batch", [("range2d", 20, 20, 3), ("cv4d", 33, 60, 2), ("growth1d", 64, 128, 2),
                                                 ("arm7", 10, 10, 300), ("range2d", 24, 24, 512),
                                                 ("range2d", 24, 24, 513)])
def test_batched_step_as_the_vector_alu_kernel(name, n, n_prev, batch, dt):
    """Drawn particles, a forward-recursion row with duplicated previous
    particles (exact ties: lowest index, tie flags), strided outputs; with no
    iterations the rows are equal, after some the particles agree."""
    announce("small set batch", name, n, n_prev, batch, dt)
    wl, desc, xp, x, z, mask = _svgd_case(name, n, n_prev, 43, dt)
    xp[n_prev // 2:] = xp[: n_prev - n_prev // 2]
    td, model, W = tdt(dt), smsq.Model(desc), max(n, n_prev) + 3
    rep = lambda a, t: dev(np.repeat(a[None], batch, 0), t)
    phi_prev = torch.zeros((batch, W), dtype=td, device=DEV)[:, :n_prev]
    for L in (0, 8):
        res = {}
        for sk in ("auto", "valu"):
            xg = torch.zeros((batch, n, desc.d), dtype=td, device=DEV)
            phi = torch.zeros((batch, W), dtype=td, device=DEV)[:, :n]
            psi = torch.full((batch, W), -7, dtype=torch.int32, device=DEV)[:, :n]
            fl = torch.full((batch, W), 9, dtype=torch.uint8, device=DEV)[:, :n]
            ws = smsq.workspace()
            smsq.batch_step(model, dt, 2, rep(xp, td), phi_prev, rep(z, td),
                            None if mask is None else rep(mask, torch.uint8), xg,
                            smsq.opts(L, 1e-5 if name == "arm7" else 0.005, step_kernel=sk), seed=11, phi=phi,
                            psi=psi, flags=fl, tie_tol=1e-6, ws=ws)
            assert smsq.device_status(ws) == smsq.OK
            res[sk] = [host(v) for v in (xg, phi, psi, fl)]
        (xa, pa, ia, fa), (xv, pv, iv, fv) = res["auto"], res["valu"]
        assert np.linalg.norm(xa - xv) <= TOL_X[dt] * np.linalg.norm(xv)
        if L == 0:
            assert np.array_equal(xa, xv) and np.array_equal(ia, iv) and np.array_equal(fa, fv)
            assert fa.all() and (ia < n_prev // 2 + n_prev % 2).all()
            assert np.abs(pa - pv).max() <= (1e-5 if dt == "f32" else 1e-13) * max(1.0, np.abs(pv).max())
