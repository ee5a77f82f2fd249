"""The 128 x 4 tiles of more than four mechanisms against the one-thread-per-
point kernels, bit for bit, at their edges; and grids on either side of the
rules that order the tiles (bands, shifted bands, plain order)."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu


def _run(prob, state, config, monkeypatch, steps):
    from paper_2106_11476_amd import fw2
    if config is None:
        monkeypatch.delenv("FW2_KERNEL_CONFIG", raising=False)
    else:
        monkeypatch.setenv("FW2_KERNEL_CONFIG", config)
    dom = fw2.from_problem(prob, device="cuda:0", cap_steps=steps)
    dom.write_fields(state)
    dom.step(steps)
    out = dict(dom.read_fields(), trace=dom.trace.cpu().numpy())
    dom.destroy_domain()
    return out


def _problem(shape, L, scheme, local, n_src):
    rng = np.random.default_rng(L)
    nb = min(4, min(shape) // 2)
    prob = W.random_medium(shape, L, 3, seed=5, nb=nb, ntr=nb // 2)
    prob.relax_scheme, prob.stencil_mode = scheme, local
    prob.src_idx = rng.choice(prob.npts, n_src, replace=False).astype(np.int64)
    prob.src_sig = rng.integers(0, 2, n_src).astype(np.int32)
    prob.src_w = rng.uniform(0.5, 1.0, n_src).astype(np.float32)
    prob.signals = (1e4 * rng.standard_normal((2, 2))).astype(np.float32)        # ends within the run
    prob.rcv_idx = rng.choice(prob.npts, min(9, prob.npts), replace=False).astype(np.int64)
    return prob


@pytest.mark.parametrize("shape", [(128, 4), (129, 5), (127, 9), (257, 3), (1, 6), (384, 64)])
@pytest.mark.parametrize("L,scheme,local", [(5, 1, 0), (6, 0, 1), (7, 0, 0), (8, 1, 1)])
def test_wide_tiles_at_their_edges(shape, L, scheme, local, monkeypatch):
    _torch()
    prob = _problem(shape, L, scheme, local, min(40, shape[0] * shape[1]))
    state = dict(zip(("p", "v", "psi1", "psi2"), W.random_state(2, L, shape, seed=3)))
    _say("128 x 4 tiles", shape, "L", L)
    ref, got = (_run(prob, state, c, monkeypatch, 3) for c in ("0,64,8", "5,64,4"))
    for k in ref:
        assert np.array_equal(ref[k], got[k]), k


# shifted bands, bands, and past 1 GiB of arrays (the first and the last grid
# on either side, and a wide one) plain order
@pytest.mark.parametrize("shape,L", [((2048, 2048), 5), ((1900, 2252), 5), ((2048, 2112), 5), ((3072, 3882), 4),
                                     ((3072, 3883), 4), ((12000, 1700), 2), ((2048, 3400), 8)])
def test_orders_of_tiles_equal_the_per_point_kernels(shape, L, monkeypatch):
    _torch()
    prob = _problem(shape, L, 1, 0, 30)
    state = dict(zip(("p", "v", "psi1", "psi2"), W.random_state(2, L, shape, seed=4)))
    _say("order of tiles", shape, "L", L)
    ref, got = (_run(prob, state, c, monkeypatch, 3) for c in ("0,64,8", None))
    for k in ref:
        assert np.array_equal(ref[k], got[k]), k


@pytest.mark.parametrize("shape,L,banded", [((300, 200, 100), 6, "3,64,13"), ((330, 220, 126), 4, "3,64,16")])
def test_orders_of_3d_tiles_give_the_same_bits(shape, L, banded, monkeypatch):
    """Past 1 GiB of arrays and with a tile count that is no multiple of 8, the
    3D sweeps take their tiles in plain order; 5 x 25 x 8 and 6 x 28 x 8 tiles
    go in bands."""
    _torch()
    prob = _problem(shape, L, 1, 0, 30)
    state = dict(zip(("p", "v", "psi1", "psi2"), W.random_state(3, L, shape, seed=4)))
    _say("order of 3D tiles", shape, "L", L)
    ref, got, plain = (_run(prob, state, c, monkeypatch, 3) for c in (banded, None, "3,64,11"))
    for k in ref:
        assert np.array_equal(ref[k], got[k]) and np.array_equal(ref[k], plain[k]), k
