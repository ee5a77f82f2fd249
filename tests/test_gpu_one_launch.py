"""One-launch steps of small 2D grids (both phases, sources and receivers in
one kernel, out of place) against the two-phase kernels, bit for bit: the
per-point arithmetic is the same, only the tiles differ."""
import numpy as np
import pytest

import workloads as W
from paper_2106_11476_amd import fw2

pytestmark = pytest.mark.gpu


def _problem(shape, L, scheme, local, n_src, seed=5):
    rng = np.random.default_rng(seed + L)
    nb = min(4, min(shape) // 2)
    prob = W.random_medium(shape, L, 3, seed=seed, nb=nb, ntr=nb // 2)
    prob.relax_scheme, prob.stencil_mode = scheme, local
    if n_src:
        prob.src_idx = rng.choice(prob.npts, n_src, replace=False).astype(np.int64)
        prob.src_sig = rng.integers(0, 2, n_src).astype(np.int32)
        prob.src_w = rng.uniform(0.5, 1.0, n_src).astype(np.float32)
        prob.signals = (1e4 * rng.standard_normal((2, 6))).astype(np.float32)   # ends within the run
    prob.rcv_idx = rng.choice(prob.npts, min(9, prob.npts), replace=False).astype(np.int64)
    return prob


def _run(prob, config, monkeypatch, chunk, steps, state):
    if config is None:
        monkeypatch.delenv("FW2_KERNEL_CONFIG", raising=False)
    else:
        monkeypatch.setenv("FW2_KERNEL_CONFIG", config)
    dom = fw2.from_problem(prob, device="cuda:0", cap_steps=sum(steps))
    dom.write_fields(dict(zip(("p", "v", "psi1", "psi2"), state)))
    dom.set_graph_chunk(chunk)
    for n in steps:
        dom.step(n)
    out = dict(dom.read_fields(fw2.FIELD_ALL), trace=dom.trace.cpu().numpy())
    at = dom.current_step()
    # the same steps out of place, from the state they started at
    dom.write_fields(dict(zip(("p", "v", "psi1", "psi2"), state)))
    dom.set_current_step(0)
    first, blocks = dom.new_state_buffer(), dom.new_state_buffer(5)
    dom.save_state(first)
    dom.step_into(5, first, blocks)
    out["into"] = blocks.cpu().numpy()
    dom.destroy_domain()
    return out, at


# tile edges (64 columns; 8 and 16 rows) and grids below the stencil's reach
SHAPES = [(64, 16), (65, 17), (63, 49), (128, 24), (200, 77), (5, 3), (1, 9), (130, 1)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("L,scheme,local", [(1, 1, 0), (2, 1, 0), (2, 0, 1), (3, 0, 0), (4, 1, 1)])
def test_one_launch_steps_equal_two_phases(shape, L, scheme, local, monkeypatch):
    prob = _problem(shape, L, scheme, local, n_src=min(40, shape[0] * shape[1]))
    state = W.random_state(2, L, shape, seed=L)
    ref, at = _run(prob, "0,64,8", monkeypatch, 4, (7, 1, 4), state)
    for config in ("4,64,8", "4,64,16", "5,64,8", None):
        for chunk in (4, 3, 0):                     # graphs of even and odd length, direct launches
            got, at2 = _run(prob, config, monkeypatch, chunk, (7, 1, 4), state)
            assert at2 == at == 12
            for k in ref:
                assert np.array_equal(ref[k], got[k]), (config, chunk, k)


@pytest.mark.parametrize("n_src", [0, 4096, 4097])
def test_source_counts_at_the_one_launch_limit(n_src, monkeypatch):
    """Up to 4096 sources are added by the tiles; one more takes the two phases."""
    shape = (140, 90)
    prob = _problem(shape, 2, 1, 0, n_src)
    state = W.random_state(2, 2, shape, seed=8)
    ref, _ = _run(prob, "0,64,8", monkeypatch, 4, (9,), state)
    got, _ = _run(prob, None, monkeypatch, 4, (9,), state)
    for k in ref:
        assert np.array_equal(ref[k], got[k]), k


def test_removing_and_adding_sources_and_receivers(monkeypatch):
    """Captured one-launch graphs follow a change of sources and receivers."""
    prob = _problem((90, 70), 2, 1, 0, 30)
    outs = []
    for config in ("0,64,8", None):
        if config is None:
            monkeypatch.delenv("FW2_KERNEL_CONFIG", raising=False)
        else:
            monkeypatch.setenv("FW2_KERNEL_CONFIG", config)
        dom = fw2.from_problem(prob, device="cuda:0", cap_steps=64)
        dom.set_graph_chunk(4)
        dom.step(8)
        dom.add_source(prob.src_idx[:5] + 1, prob.src_sig[:5], prob.src_w[:5], np.ones((2, 30), np.float32))
        dom.step(8)
        trace = dom.trace.clone()
        dom.add_receivers(prob.rcv_idx[:3], 64)
        dom.step(9)
        outs.append((trace.cpu().numpy(), dom.trace.cpu().numpy(), dom.read_fields(fw2.FIELD_P)["p"]))
        dom.destroy_domain()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("shape,L", [((1100, 900), 4), ((1900, 1700), 4), ((1030, 1000), 2)])
def test_grids_around_the_cache_limits_equal_the_per_point_kernels(shape, L, monkeypatch):
    """Two phases with the memory variables kept in the cache (217 MB of arrays
    at most), streamed past it (300 MB), and one launch of many tiles."""
    prob = _problem(shape, L, 1, 0, 5)
    state = W.random_state(2, L, shape, seed=2)
    ref, _ = _run(prob, "0,64,8", monkeypatch, 4, (3,), state)
    got, _ = _run(prob, None, monkeypatch, 4, (3,), state)
    for k in ref:
        assert np.array_equal(ref[k], got[k]), k


@pytest.mark.parametrize("shape,L,scheme,local,config", [
    ((65, 17), 5, 1, 0, "5,64,4"), ((63, 5), 6, 0, 1, "5,64,4"), ((130, 3), 7, 0, 0, "5,64,4"),
    ((64, 8), 8, 1, 1, "5,64,4"), ((2011, 1203), 8, 1, 0, None)])
def test_four_row_tiles_equal_the_per_point_kernels(shape, L, scheme, local, config, monkeypatch):
    """More than four mechanisms: tiles of four rows at their edges, and chosen
    by a grid whose arrays (377 MB) pass the cache."""
    prob = _problem(shape, L, scheme, local, 6)
    state = W.random_state(2, L, shape, seed=3)
    ref, _ = _run(prob, "0,64,8", monkeypatch, 4, (3,), state)
    got, _ = _run(prob, config, monkeypatch, 4, (3,), state)
    for k in ref:
        assert np.array_equal(ref[k], got[k]), k
