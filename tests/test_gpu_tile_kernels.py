"""The 2D kernels of LDS tiles, each chosen by name, against the FP64 oracle
(both schemes, global and per-point stencil weights, tiles that overhang the
grid) and, where a grid's size decides between them, against the
one-thread-per-point kernels bit for bit."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import _say, _state, compare, gpu_run, oracle_run

pytestmark = pytest.mark.gpu

CASES = [((70, 45), 2, 1), ((257, 131), 4, 1), ((131, 90), 3, 0), ((64, 16), 1, 0), ((65, 17), 2, 0)]
MANY = [((70, 45), 5, 1), ((131, 40), 6, 0), ((64, 49), 8, 1), ((130, 33), 7, 0)]


@pytest.mark.parametrize("config", ["4,64,8", "4,64,16", "5,64,8", "5,64,16"])
@pytest.mark.parametrize("shape,L,scheme", CASES)
@pytest.mark.parametrize("local", [0, 1])
def test_tile_kernels_match_oracle(monkeypatch, config, shape, L, scheme, local):
    monkeypatch.setenv("FW2_KERNEL_CONFIG", config)
    _check(config, shape, L, scheme, local)


@pytest.mark.parametrize("config", ["5,64,4", "5,64,8", "5,64,16"])
@pytest.mark.parametrize("shape,L,scheme", MANY)
@pytest.mark.parametrize("local", [0, 1])
def test_tile_kernels_of_many_mechanisms_match_oracle(monkeypatch, config, shape, L, scheme, local):
    monkeypatch.setenv("FW2_KERNEL_CONFIG", config)
    _check(config, shape, L, scheme, local)


def _check(config, shape, L, scheme, local):
    prob = W.random_medium(shape, L, 3, seed=7, nb=min(8, min(shape) // 2), ntr=min(5, min(shape) // 3))
    prob.relax_scheme, prob.stencil_mode = scheme, local
    st = _state(prob, 13)
    _say("tiles", config, shape, "L", L, "scheme", scheme, "local", local)
    f, tr, _ = gpu_run(prob, 12, state=st)
    ref, rtr = oracle_run(prob, 12, state=st)
    compare(f, tr, ref, rtr, "tiles %s %s" % (config, shape), prob=prob)


# (shape, L): the last grid on one side of a limit and the first on the other.
# 1500 columns are rows of 1536: L = 4, 22 arrays, the memory variables kept in
# the cache up to 240 MiB; L = 2, two state blocks and the medium, 25 arrays,
# one launch a step up to 240 MiB; L = 4 with at most 256 tiles of 64 x 16.
LIMITS = [((1500, 1853), 4), ((1500, 1854), 4), ((1500, 1630), 2), ((1500, 1631), 2), ((1024, 256), 4), ((1024, 257), 4)]


@pytest.mark.parametrize("shape,L", LIMITS)
def test_grids_at_the_size_limits_equal_the_per_point_kernels(monkeypatch, shape, L):
    from paper_2106_11476_amd import fw2
    prob = W.random_medium(shape, L, 3, seed=5, nb=6, ntr=4)
    st = W.random_state(2, L, shape, seed=2)
    _say("size limits", shape, "L", L)
    out = []
    for config in ("0,64,8", None, "5,64,16"):
        if config is None:
            monkeypatch.delenv("FW2_KERNEL_CONFIG", raising=False)
        else:
            monkeypatch.setenv("FW2_KERNEL_CONFIG", config)
        dom = fw2.Domain(prob, device="cuda:0")
        dom.write_fields(dict(zip(("p", "v", "psi1", "psi2"), st)))
        dom.step(3)
        out.append(dom.read_fields())
        dom.destroy_domain()
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k]) and np.array_equal(out[0][k], out[2][k]), k
