"""Domains with and without the second state block of the one-launch step:
equal bits, and a server whose budget holds the requests' single blocks takes
them."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import _say, _state, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,L,scheme,local", [((97, 131), 2, 1, 0), ((64, 48), 4, 0, 1), ((200, 77), 1, 1, 0)])
def test_without_the_second_block_the_same_bits(shape, L, scheme, local):
    torch = _torch()
    from paper_2106_11476_amd import fw2
    prob = W.random_medium(shape, L, 3, seed=L, nb=6, ntr=4)
    prob.relax_scheme, prob.stencil_mode = scheme, local
    st = _state(prob, 5)
    _say("second block", shape, "L", L)
    out = []
    for second in (True, False):
        dom = fw2.Domain(prob, device="cuda:0", second_block=second)
        assert dom.workspace_bytes == fw2.workspace_bytes(prob, second_block=second)
        dom.write_fields(st)
        for n in (2, 1, 70):
            dom.step(n)
        blocks, first = dom.new_state_buffer(3), dom.new_state_buffer()
        dom.save_state(first)
        dom.step_into(3, first, blocks)
        torch.cuda.synchronize()
        out.append((dom.read_fields(), blocks.cpu().numpy(), first.cpu().numpy()))
        dom.destroy_domain()
    (a, ia, fa), (b, ib, fb) = out
    assert np.array_equal(ia, ib) and np.array_equal(fa, fb)
    for k in a:
        assert np.array_equal(a[k], b[k]), k


def _request(shape, seed):
    from paper_2106_11476_amd import serve
    p = W.random_medium(shape, 2, 2, seed=seed, nb=6, ntr=4)
    p.src_idx = np.array([p.npts // 2], np.int64)
    p.src_sig, p.src_w = np.zeros(1, np.int32), np.ones(1, np.float32)
    p.signals = W.gaussian_pulse(40, p.dt, 3e6, 3, 1e5)[None]
    p.rcv_idx = np.arange(3, dtype=np.int64) + p.npts // 2
    return serve.Request(rid=seed, problem=p, n_steps=90)


def _check_traces(reqs):
    torch = _torch()
    from paper_2106_11476_amd import fw2
    for r in reqs:
        solo = fw2.from_problem(r.problem, device="cuda:0", cap_steps=90)
        solo.step(90)
        torch.cuda.synchronize()
        assert np.array_equal(solo.trace.cpu().numpy(), r.trace)
        solo.destroy_domain()


def test_a_budget_of_single_blocks_serves_the_requests():
    """Requests of one batch and a larger one stepped alone, within a budget of
    exactly their single blocks."""
    _torch()
    from paper_2106_11476_amd import serve
    reqs = [_request(s, k) for k, s in enumerate([(128, 128), (120, 90), (320, 260)])]
    _say("served within single blocks")
    budget = sum(serve.footprint_bytes(r.problem, 90) for r in reqs)
    srv = serve.Server(budget_bytes=budget, max_active=4, solo_points=320 * 260)
    stats = srv.run(reqs)
    srv.close()
    assert stats.completed == 3 and stats.peak_bytes <= budget
    _check_traces(reqs)


@pytest.mark.parametrize("short", [0, 1])
def test_a_request_stepped_alone_takes_the_second_block_where_the_budget_has_it(short):
    _torch()
    from paper_2106_11476_amd import fw2, serve
    r = _request((320, 260), 7)
    _say("solo request,", short, "bytes short of a second block")
    extra = fw2.workspace_bytes(r.problem, second_block=True) - fw2.workspace_bytes(r.problem)
    single = serve.footprint_bytes(r.problem, 90)
    srv = serve.Server(budget_bytes=single + extra - short, max_active=4, solo_points=1)
    stats = srv.run([r])
    srv.close()
    assert stats.completed == 1 and extra > 0
    assert r.footprint == single + (0 if short else extra) and stats.peak_bytes == r.footprint
    _check_traces([r])
