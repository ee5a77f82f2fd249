"""2D reverse steps from LDS tiles at the tiles' edges (64 columns; 8 rows up
to two mechanisms, 16 above) and at the tiles' source limit, against the
oracle's FP64 adjoint.

The bar is that of the other gradient tests (5e-4 in relative L2 and in
max-abs of the peak): the gradient sums products of the forward and the
adjoint state, each within the FP32 forward error."""
import numpy as np
import pytest

import workloads as W
from oracle import adjoint as oadj
from oracle import solver

pytestmark = pytest.mark.gpu


def _problem(shape, L, n, n_src):
    rng = np.random.default_rng(shape[0] + L)
    prob = W.random_medium(shape, L, 3, seed=11, nb=3, ntr=2)
    prob.n_steps = n
    prob.fd_r = float(prob.c.max()) * prob.dt / prob.h
    prob.pml_cp = float(prob.c.max())
    prob.src_idx = rng.choice(prob.npts, n_src, replace=False).astype(np.int64)
    prob.src_sig = np.zeros(n_src, np.int32)
    prob.src_w = rng.uniform(0.2, 1.0, n_src).astype(np.float32)
    prob.signals = W.gaussian_pulse(n, prob.dt, 2e7, 3, 2e5)[None]
    prob.rcv_idx = rng.choice(prob.npts, 12, replace=False).astype(np.int64)
    return prob


def _check(prob, n, K):
    import torch
    from paper_2106_11476_amd import adjoint
    pert = W.Problem(**{k: getattr(prob, k) for k in prob.__dataclass_fields__})
    pert.c = np.minimum(prob.c * 1.01, prob.c.max()).astype(np.float32)
    obs = solver.run(pert, n)[1]
    c = torch.tensor(np.asarray(prob.c, np.float64), requires_grad=True)
    J = adjoint.misfit(c, torch.tensor(np.asarray(obs, np.float32), device="cuda:0"), prob, n, checkpoint_every=K)
    J.backward()
    J_ref, g_ref, _ = oadj.misfit_and_gradient(prob, obs, n)
    d = c.grad.numpy() - g_ref
    assert abs(J.item() - J_ref) <= 1e-3 * J_ref
    assert np.linalg.norm(d) <= 5e-4 * np.linalg.norm(g_ref)
    assert np.abs(d).max() <= 5e-4 * np.abs(g_ref).max()


@pytest.mark.parametrize("shape,L", [((64, 8), 2), ((65, 17), 1), ((63, 16), 3), ((128, 33), 4), ((129, 15), 8),
                                     ((7, 70), 2)])
def test_gradient_at_tile_edges(shape, L):
    _check(_problem(shape, L, 40, 3), 40, 7)


@pytest.mark.parametrize("n_src", [4096, 4097])
def test_gradient_at_the_source_limit(n_src):
    _check(_problem((90, 60), 2, 24, n_src), 24, 24)
