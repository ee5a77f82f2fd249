"""A batch follows its domains' own step counters: a member that is reloaded,
set to another step, stepped alone or replayed from a caller's graph between
two batch calls goes on from where its counter stands, bit for bit as it does
alone, without a new set_domains."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu

N = 60                       # steps of every member


def _problem(shape, L, seed):
    p = W.random_medium(shape, L, 2, seed=seed, nb=6, ntr=4)
    rng = np.random.default_rng(seed)
    p.src_idx = np.unique(rng.integers(0, p.npts, 6)).astype(np.int64)
    p.src_sig = np.zeros(p.src_idx.size, np.int32)
    p.src_w = np.ones(p.src_idx.size, np.float32)
    p.signals = (1e4 * rng.standard_normal((1, N))).astype(np.float32)      # every step its own sample
    p.rcv_idx = rng.integers(0, p.npts, 5).astype(np.int64)
    return p


PROBLEMS = [((90, 70), 2, 3), ((70, 45), 6, 4), ((130, 33), 3, 5)]


def _run(batched, script, stream):
    """The script's calls on every domain; `step` runs in a batch that is set
    once, or domain by domain."""
    from paper_2106_11476_amd import fw2
    doms = [fw2.from_problem(_problem(*a), device="cuda:0", stream=stream, cap_steps=N) for a in PROBLEMS]
    start = [d.new_state_buffer() for d in doms]
    for d, s in zip(doms, start):
        d.save_state(s)
    batch = None
    if batched:
        batch = fw2.Batch(max_domains=4, stream=stream)
        batch.set_domains(doms, [N] * len(doms))

    def step(n):
        if batched:
            batch.step(n)
        else:
            for d in doms:
                d.step(min(n, N - d.current_step()))
        stream.synchronize()

    script(doms, start, step)
    stream.synchronize()
    out = []
    for d in doms:
        out.append((d.current_step(), d.trace.cpu().numpy(), d.read_fields(fw2.FIELD_ALL)))
    if batched:
        batch.destroy()
    for d in doms:
        d.destroy_domain()
    return out


def _restart_finished(doms, start, step):
    step(N)
    for d, s in zip(doms, start):
        d.load_state(s, 0)
        d.trace.zero_()
    step(N)


def _restart_midway(doms, start, step):
    step(37)
    doms[1].load_state(start[1], 20)
    step(40)


def _set_counter(doms, start, step):
    step(10)
    doms[0].set_current_step(33)
    doms[2].set_current_step(2)
    step(40)


def _step_alone(doms, start, step):
    step(9)
    doms[0].step(5)
    doms[1].step(32)
    step(34)


@pytest.mark.parametrize("script", [_restart_finished, _restart_midway, _set_counter, _step_alone])
def test_members_moved_between_batch_calls_equal_solo_runs(script):
    torch = _torch()
    _say("batch members moved:", script.__name__)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ref = _run(False, script, stream)
        got = _run(True, script, stream)
    for (n0, t0, f0), (n1, t1, f1) in zip(ref, got):
        assert n0 == n1
        assert np.abs(t0).max() > 0 and np.array_equal(t0, t1)
        for k in f0:
            assert np.array_equal(f0[k], f1[k]), k


def test_member_replayed_from_a_callers_graph_joins_at_its_counter():
    """The caller captures ten steps and replays them three times: the device
    counter stands at 30, the host's count at 10.  The batch stops the member
    at its n_steps by the counter."""
    torch = _torch()
    from paper_2106_11476_amd import fw2
    _say("batch member stepped by a caller's graph")
    stream = torch.cuda.Stream()
    prob = _problem(*PROBLEMS[0])
    solo = fw2.from_problem(prob, device="cuda:0", stream=stream, cap_steps=N)
    solo.step(N)
    dom = fw2.from_problem(prob, device="cuda:0", stream=stream, cap_steps=N)
    dom.set_graph_chunk(0)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
        dom.step(10)
    with torch.cuda.stream(stream):
        for _ in range(3):
            graph.replay()
    stream.synchronize()
    batch = fw2.Batch(max_domains=2, stream=stream)
    batch.set_domains([dom], [N])
    batch.step(50)                              # 30 to go, idle past them
    stream.synchronize()
    assert torch.equal(dom.trace, solo.trace)
    a, b = dom.read_fields(), solo.read_fields()
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    batch.destroy()
    dom.destroy_domain()
    solo.destroy_domain()
