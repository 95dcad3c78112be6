"""Which step kernel the automatic choice takes on either side of its limits.
Kernels sum in different orders, so a step's bits tell: those of the automatic
choice are those of the kernel it takes."""
import numpy as np
import pytest
import torch

from paper_2312_08684_amd import scenarios as S
from paper_2312_08684_amd import smsq
from test_gpu_parity import DEV, announce

pytestmark = pytest.mark.gpu


def particles(name, batch, n, dtype, step_kernel, iters=4):
    """The second step's particles of a batch of sequences."""
    wl = S.make_workload(name, B=2, seed=1500, T=2, n=n, n_iter=iters)
    td = torch.float32 if dtype == "f32" else torch.float64
    rep = lambda a, t: torch.tensor(np.ascontiguousarray(a[np.arange(batch) % 2]), dtype=t, device=DEV)
    model = smsq.Model(wl.model)
    mask = None if wl.mask is None else rep(wl.mask, torch.uint8)
    parts = torch.zeros((batch, 2, n, wl.model.d), dtype=td, device=DEV)
    ws = smsq.workspace(model.workspace_size(dtype, batch, 2, n))
    smsq.run_batch(model, dtype, rep(wl.x0, td), rep(wl.z, td), mask, n,
                   smsq.opts(iters, wl.opts.step, step_kernel=step_kernel), 7, particles=parts, ws=ws)
    assert smsq.device_status(ws) == smsq.OK
    return parts[:, 1]


# several workgroups a sequence: at least 2^19 n^-2 times the part of the 256
# compute units that they fill
@pytest.mark.parametrize("n,batch,several", [(448, 4, False), (512, 1, True), (512, 16, True), (512, 17, False),
                                             (512, 64, False), (640, 64, True), (768, 64, True), (1024, 64, True),
                                             (1024, 65, False)])
def test_several_workgroups(n, batch, several):
    announce("routes", n, batch, several)
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("limits of 256 compute units")
    auto = particles("range2d", batch, n, "f32", "auto")
    assert torch.equal(auto, particles("range2d", batch, n, "f32", "mfma")) != several
    assert not several or torch.equal(auto, particles("range2d", batch, n, "f32", "coop"))


# small sets: up to one sequence a compute unit, or two
@pytest.mark.parametrize("name,n,batch,dtype,other", [("range2d", 24, 512, "f32", None), ("range2d", 24, 513, "f32", "wave"),
                                                      ("cv4d", 48, 256, "f32", None), ("cv4d", 48, 257, "f32", "mfma"),
                                                      ("cv4d", 40, 512, "f64", None), ("cv4d", 40, 513, "f64", "valu")])
def test_small_sets(name, n, batch, dtype, other):
    announce("routes", name, n, batch, dtype, other)
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("limits of 256 compute units")
    auto = particles(name, batch, n, dtype, "auto")
    for sk in ("wave", "mfma", "valu"):
        if sk == "mfma" and dtype == "f64" or sk == "wave" and n > 32:
            continue
        assert torch.equal(auto, particles(name, batch, n, dtype, sk)) == (sk == other), sk
