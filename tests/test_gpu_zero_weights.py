"""Sources of weight exactly zero (a log-weight of minus infinity) in the steps
that weigh the previous particles: blocks, whole shares of a wave and all but one
source, on the matrix cores and in the small-set kernel, whose first chunk of 64
sources then holds none.  Teacher-forced against the oracle with the tolerances
of those steps."""
import numpy as np
import pytest

from test_gpu_parity import _compare_svgd, _svgd_case, announce

pytestmark = pytest.mark.gpu


def log_weights(n_prev, zero):
    w = np.random.default_rng(9).dirichlet(np.ones(n_prev))
    for lo, hi in zero:
        w[lo:hi] = 0.0
    with np.errstate(divide="ignore"):
        return np.log(w / w.sum()).astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("name,step", [("range2d", 0.005), ("cv4d", 0.005), ("arm7", 1e-5)])
@pytest.mark.parametrize("n", [64, 100, 600])
@pytest.mark.parametrize("zero", [[(0, 40), (96, 200)], [(0, 160)], [(128, 300)], [(0, 150), (151, 300)]])
def test_matrix_step(zero, n, name, step):
    announce("zero weights, matrix step", zero, n, name)
    wl, desc, xp, x, z, mask = _svgd_case(name, n, 300, 90, "f32")
    _compare_svgd(desc, "f32", xp, log_weights(300, zero), z, mask, x, 8, step, step_kernel="mfma")


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("name", ["range2d", "cv4d"])
@pytest.mark.parametrize("n_prev,zero", [(100, [(0, 64)]), (128, [(64, 128)]), (70, [(0, 69)]), (20, [(1, 20)]),
                                         (64, [(3, 60)])])
def test_small_sets(n_prev, zero, name, dt):
    announce("zero weights, small sets", n_prev, zero, name, dt)
    wl, desc, xp, x, z, mask = _svgd_case(name, 40, n_prev, 91, dt)
    _compare_svgd(desc, dt, xp, log_weights(n_prev, zero), z, mask, x, 10, 0.005)
