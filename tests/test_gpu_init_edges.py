"""Proposal network at the edges of its kernels' tiles: batches around the 16
rows of a workgroup and the 8 products in flight of a weight gradient (128
rows), particle counts around the 256 of a likelihood chunk, against the CPU
oracle (oracle/init_mlp.py).

Forward and gradients: the oracle applies the same BF16 roundings and
accumulates in FP64.  FP32 sums of up to 320 products differ from it by about
1e-6, but may round one operand of the next product to the other BF16
neighbour: 2^-8 of that element, 4e-3 of the largest gradient at most.  Mixture
NLL: FP32 against FP64, 1e-4 as at the other sizes."""
import numpy as np
import pytest
import torch

from oracle import init_mlp as M
from paper_2312_08684_amd import scenarios as S
from paper_2312_08684_amd import smsq

pytestmark = pytest.mark.gpu

FLIP = 2.0 ** -8


def _rel(a, b):
    return np.abs(np.asarray(a, np.float64) - b).max() / max(1e-30, np.abs(b).max())


def _check(mlp, P, F, dout):
    out = mlp.forward(torch.tensor(F, device="cuda")).cpu().numpy()
    ref, cache = M.forward(P, F.astype(np.float64), bf16=True)
    assert _rel(out, ref) <= FLIP
    mlp.backward(torch.tensor(dout, device="cuda"))
    G, R = mlp.grads().cpu().numpy(), M.backward(cache, dout.astype(np.float64), bf16=True)
    for name, lo, hi in [("W1", M.OFF_W1, M.OFF_B1), ("b1", M.OFF_B1, M.OFF_W2), ("W2", M.OFF_W2, M.OFF_B2),
                         ("b2", M.OFF_B2, M.OFF_W3), ("W3", M.OFF_W3, M.OFF_B3), ("b3", M.OFF_B3, M.N_PARAMS)]:
        assert _rel(G[lo:hi], R[lo:hi]) <= FLIP, name


@pytest.mark.parametrize("batch", [1, 15, 16, 17, 127, 128, 129, 145, 300])
def test_network_at_batch_edges(batch):
    rng = np.random.default_rng(batch)
    P = rng.normal(scale=0.15, size=M.N_PARAMS).astype(np.float32).astype(np.float64)
    mlp = smsq.InitMLP(seed=1, max_batch=300)
    mlp.set_params(torch.tensor(P, dtype=torch.float32, device="cuda"))
    # a larger batch before: nothing of its rows may count
    mlp.forward(torch.full((300, M.FEAT), 3e4, device="cuda"))
    mlp.backward(torch.full((300, M.OUT), float("inf"), device="cuda"))
    _check(mlp, P, rng.normal(size=(batch, M.FEAT)).astype(np.float32),
           rng.normal(size=(batch, M.OUT)).astype(np.float32))


def _set(n, count, seed):
    rng = np.random.default_rng(seed)
    wl = S.make_workload("cv4d", B=1, seed=seed, n=64, T=2, n_iter=1)
    model = smsq.Model(wl.model)
    z = torch.tensor(wl.z[0][1], dtype=torch.float32, device="cuda")
    mask = torch.tensor(wl.mask[0][1], dtype=torch.uint8, device="cuda") if wl.mask is not None else None
    t = lambda *s: torch.tensor(rng.normal(size=s), dtype=torch.float32, device="cuda")
    ex = [{"model": 0, "t": 2, "x_prev": t(70, 4), "phi_prev": t(70), "z": z, "z_mask": mask, "particles": t(n, 4),
           "seed": 5, "seq": k} for k in range(count)]
    return model, ex, smsq.InitSet([model], ex)


@pytest.mark.parametrize("n", [1, 63, 65, 255, 256, 257, 513])
def test_mixture_nll_at_chunk_edges(n):
    model, ex, iset = _set(n, 3, n)
    mlp = smsq.InitMLP(seed=0, max_batch=4)
    _, A, Sc = mlp.features(iset)
    rng = np.random.default_rng(n)
    out = rng.normal(scale=0.5, size=(len(ex), M.OUT)).astype(np.float32)
    out[1, 8] = 5.0   # a log-scale past its clamp
    loss, dout = iset.nll(torch.tensor(out, device="cuda"), A, Sc, gscale=1.0)
    loss, dout = loss.cpu().numpy(), dout.cpu().numpy()
    for k, q in enumerate(ex):
        lr, gr = M.mixture_nll(out[k].astype(np.float64), A[k].cpu().numpy(), Sc[k].cpu().numpy(),
                               q["particles"].cpu().numpy())
        assert abs(loss[k] - lr) <= 1e-4 * max(1.0, abs(lr))
        assert np.abs(dout[k] - gr).max() <= 1e-4 * max(1.0, np.abs(gr).max())


def test_training_keeps_every_copy_of_the_weights():
    """After training steps the products use the parameters that were stepped
    to, in both orders of the weights."""
    model, ex, iset = _set(40, 37, 3)
    mlp = smsq.InitMLP(seed=2, max_batch=64)
    before = mlp.params().cpu().numpy().copy()
    for _ in range(3):
        mlp.train_step(iset, 0, 37, 1e-2)
    P = mlp.params().cpu().numpy().astype(np.float64)
    assert np.abs(P - before).max() > 1e-3
    rng = np.random.default_rng(1)
    _check(mlp, P, rng.normal(size=(37, M.FEAT)).astype(np.float32),
           rng.normal(size=(37, M.OUT)).astype(np.float32))
