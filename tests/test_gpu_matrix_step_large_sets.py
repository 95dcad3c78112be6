"""Matrix-core steps after previous sets too large for one compute unit's LDS
beside the particles (d >= 4), taken in chunks: against the oracle, on the
matrix cores at every size that FP32 tables held (their bits differ from the
vector-ALU kernel's), with weights of zero over whole chunks, the mean reading,
and the forward recursion of a batched step.  Tolerances of a teacher-forced
FP32 step."""
import numpy as np
import pytest
import torch

from paper_2312_08684_amd import smsq
from test_gpu_parity import DEV, TOL_X, _compare_svgd, _svgd_case, announce, dev, host

pytestmark = pytest.mark.gpu

STEP = {"cv4d": 0.005, "arm7": 1e-5}


def on_matrix_cores(desc, xp, z, mask, x, step):
    """Whether the automatic choice is not the vector-ALU kernel."""
    td, res = torch.float32, []
    for sk in ("auto", "valu"):
        xg = dev(x, td)
        smsq.svgd_step(smsq.Model(desc), "f32", 2, dev(xp, td), None, dev(z, td),
                       None if mask is None else dev(mask, torch.uint8), xg, smsq.opts(3, step, step_kernel=sk),
                       ws=smsq.workspace())
        res.append(xg)
    return not torch.equal(*res)


@pytest.mark.parametrize("name", ["cv4d", "arm7"])
@pytest.mark.parametrize("n,n_prev", [(64, 2000), (128, 1888), (256, 1696), (333, 1712), (640, 2000), (1024, 1376),
                                      (1024, 1089), (70, 1377), (1000, 1281), (512, 1300), (64, 2800)])
def test_sizes(n, n_prev, name):
    announce("large previous set", name, n, n_prev)
    wl, desc, xp, x, z, mask = _svgd_case(name, n, n_prev, 80, "f32")
    assert on_matrix_cores(desc, xp, z, mask, x, STEP[name])
    _compare_svgd(desc, "f32", xp, None, z, mask, x, 4, STEP[name])


@pytest.mark.parametrize("n", [100, 700])
def test_chunks_of_weight_zero(n):
    announce("large previous set, zero weights", n)
    wl, desc, xp, x, z, mask = _svgd_case("cv4d", n, 1950, 81, "f32")
    w = np.random.default_rng(8).dirichlet(np.ones(1950))
    with np.errstate(divide="ignore"):
        for lo, hi in ((0, 1000), (1000, 1950), (40, 1900)):
            v = w.copy()
            v[lo:hi] = 0.0
            log_w = np.log(v).astype(np.float32).astype(np.float64)
            _compare_svgd(desc, "f32", xp, log_w, z, mask, x, 4, STEP["cv4d"])


def test_mean_reading():
    announce("large previous set, mean reading")
    wl, desc, xp, x, z, mask = _svgd_case("arm7", 200, 1700, 82, "f32")
    _compare_svgd(desc, "f32", xp, None, z, mask, x, 4, STEP["arm7"], trans_mode=1)


@pytest.mark.parametrize("name,n,n_prev", [("cv4d", 100, 1900), ("arm7", 600, 1400)])
def test_recursion_of_a_batched_step(name, n, n_prev):
    """Rows against the vector-ALU kernel: duplicated previous particles (exact
    ties: lowest index), the second sequence weighted by its scores."""
    announce("large previous set, recursion", name, n, n_prev)
    wl, desc, xp, x, z, mask = _svgd_case(name, n, n_prev, 83, "f32")
    xp[n_prev // 2:] = xp[: n_prev - n_prev // 2]
    td, model = torch.float32, smsq.Model(desc)
    rep = lambda a, t: dev(np.repeat(a[None], 2, 0), t)
    for L in (0, 4):
        res = {}
        for sk in ("auto", "valu"):
            xg = rep(x, td)
            phi = torch.zeros((2, n_prev), dtype=td, device=DEV)[:, :n]
            psi = torch.zeros((2, n_prev), dtype=torch.int32, device=DEV)[:, :n]
            fl = torch.zeros((2, n_prev), dtype=torch.uint8, device=DEV)[:, :n]
            ws = smsq.workspace()
            smsq.batch_step(model, "f32", 2, rep(xp, td), torch.zeros((2, n_prev), dtype=td, device=DEV), rep(z, td),
                            None if mask is None else rep(mask, torch.uint8), xg, smsq.opts(L, STEP[name], step_kernel=sk),
                            init_given=True, phi=phi, psi=psi, flags=fl, tie_tol=1e-6, ws=ws)
            assert smsq.device_status(ws) == smsq.OK
            res[sk] = [host(v).astype(np.float64) for v in (xg, phi, psi, fl)]
        (xa, pa, ia, fa), (xv, pv, iv, fv) = res["auto"], res["valu"]
        assert np.linalg.norm(xa - xv) <= TOL_X["f32"] * np.linalg.norm(xv)
        if L == 0:
            # positions relative to another centre: scores to FP32 rounding of
            # squares of up to some hundreds
            assert fa.all() and (ia < n_prev // 2 + n_prev % 2).all()
            assert np.abs(pa - pv).max() <= 1e-4 * max(1.0, np.abs(pv).max())
