"""Packed fields through device memory (one launch for every selected array)
against the same call on host memory (a row copy per plane): equal values."""
import numpy as np
import pytest

import workloads as W
from paper_2106_11476_amd import fw2

pytestmark = pytest.mark.gpu

# multiples of four (four values a thread), remainders, single columns and rows
SHAPES = [(64, 12), (5, 9), (1, 7), (8, 1), (260, 3), (12, 6, 5), (7, 5, 3), (4, 1, 6), (66, 4, 1)]


def _domain(shape, L):
    prob = W.homogeneous(shape, L=L)
    dom = fw2.from_problem(prob, device="cuda:0")
    rng = np.random.default_rng(len(shape) * 100 + L)
    return dom, rng.standard_normal(dom.field_numel(fw2.FIELD_ALL)).astype(np.float32)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("offset", [0, 1])          # packed buffer on 16 bytes, or 4 past them
def test_device_fields_equal_host_fields(shape, offset):
    import torch
    for L, masks in ((1, (15, 1, 2, 4, 8, 6, 9)), (3, (15, 12))):
        dom, values = _domain(shape, L)
        for mask in masks:
            n = dom.field_numel(mask)
            buf = torch.zeros(n + offset, dtype=torch.float32, device="cuda:0")[offset:]
            buf.copy_(torch.as_tensor(values[:n]))
            dom.write_fields({k: np.zeros(s, np.float32) for k, s in dom._sizes(fw2.FIELD_ALL)})
            dom.write_fields_device(buf, mask)
            by_device = dom.read_fields(fw2.FIELD_ALL)
            dom.write_fields({k: np.zeros(s, np.float32) for k, s in dom._sizes(fw2.FIELD_ALL)})
            parts = dom.field_views(values[:n], mask)
            dom.write_fields(parts, mask)
            by_host = dom.read_fields(fw2.FIELD_ALL)
            for k in by_host:
                assert np.array_equal(by_device[k], by_host[k]), (shape, L, mask, k)
            out = torch.full((n + offset,), -1.0, dtype=torch.float32, device="cuda:0")[offset:]
            fw2._check(fw2.lib().fw2_read_fields(dom._h, mask, out.data_ptr(), fw2.DEVICE))
            host = np.concatenate([by_host[k].reshape(-1) for k, _ in dom._sizes(mask)])
            assert np.array_equal(out.cpu().numpy(), host), (shape, L, mask)
        dom.destroy_domain()


def test_device_fields_in_host_memory_go_by_copies():
    """A buffer given as device memory that no kernel should address directly
    (here pinned host memory) moves by copies, with the same values."""
    import torch
    dom, values = _domain((37, 11), 2)
    n = dom.field_numel(fw2.FIELD_ALL)
    buf = torch.as_tensor(values[:n]).pin_memory()
    fw2._check(fw2.lib().fw2_write_fields(dom._h, fw2.FIELD_ALL, buf.data_ptr(), fw2.DEVICE))
    by_device = dom.read_fields(fw2.FIELD_ALL)
    dom.write_fields(dom.field_views(values[:n], fw2.FIELD_ALL), fw2.FIELD_ALL)
    by_host = dom.read_fields(fw2.FIELD_ALL)
    for k in by_host:
        assert np.array_equal(by_device[k], by_host[k]), k
    dom.destroy_domain()


@pytest.mark.parametrize("shape,L", [((5, 9), 1), ((300, 41), 4), ((12, 6, 5), 2), ((70, 5, 3), 6)])
@pytest.mark.parametrize("offset", [0, 60, 1])      # floats past 256 bytes: on 16 bytes, on 16 bytes, not
def test_state_blocks_move_whole(shape, L, offset):
    """save_state and load_state move the block's bytes, and nothing beside it,
    whatever the buffer's alignment; captured, every replay does so again."""
    import torch
    prob = W.homogeneous(shape, L=L)
    stream = torch.cuda.Stream(device="cuda:0")
    with torch.cuda.stream(stream):
        dom = fw2.from_problem(prob, device="cuda:0", stream=stream)
        n = dom.state_bytes() // 4
        rng = np.random.default_rng(n)
        values = torch.as_tensor(rng.standard_normal(n).astype(np.float32)).to("cuda:0")
        src = torch.zeros(n + offset, device="cuda:0")[offset:]
        full = torch.full((n + 2 * 64,), -7.0, device="cuda:0")
        dst = full[offset:offset + n]
        src.copy_(values)
        dom.load_state(src, 3)
        dom.save_state(dst)
        stream.synchronize()
        assert torch.equal(dst, values) and bool((full[offset + n:] == -7.0).all())
        assert bool((full[:offset] == -7.0).all()) and dom.current_step() == 3
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            dom.load_state(src, 0)
            dom.save_state(dst)
        for k in range(3):
            src.copy_(values * (k + 2))
            full.fill_(0.0)
            graph.replay()
            stream.synchronize()
            assert torch.equal(dst, values * (k + 2)), k
    dom.destroy_domain()


@pytest.mark.parametrize("n", [(64, 64, 64), (45, 30, 70), (130, 9, 40), (33, 8, 5), (96, 40, 3)])
@pytest.mark.parametrize("L", [2, 5])
def test_3d_tile_and_march_choice_does_not_change_results(n, L, monkeypatch):
    """The tile and planes per block picked from the grid against one fixed
    choice, bit for bit (the per-point arithmetic does not depend on them)."""
    prob = W.random_medium(n, L, 3, seed=n[0] + L, nb=1, ntr=1)
    prob.src_idx = np.array([prob.npts // 2], np.int64)
    prob.src_sig, prob.src_w = np.zeros(1, np.int32), np.ones(1, np.float32)
    prob.signals = np.full((1, 4), 1e4, np.float32)
    prob.rcv_idx = np.array([0, prob.npts // 3, prob.npts - 1], np.int64)
    state = W.random_state(3, L, n, seed=3)
    got = []
    for config in (None, "3,64,64"):
        if config is None:
            monkeypatch.delenv("FW2_KERNEL_CONFIG", raising=False)
        else:
            monkeypatch.setenv("FW2_KERNEL_CONFIG", config)
        dom = fw2.from_problem(prob, device="cuda:0", cap_steps=5)
        dom.write_fields(dict(zip(("p", "v", "psi1", "psi2"), state)))
        dom.step(5)
        f = dom.read_fields(fw2.FIELD_ALL)
        got.append((f, dom.trace.cpu().numpy()))
        dom.destroy_domain()
    for k in got[0][0]:
        assert np.array_equal(got[0][0][k], got[1][0][k]), k
    assert np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("shape,L", [((70, 21, 30), 2), ((40, 33, 17), 3), ((66, 9, 40), 6)])
def test_3d_sources_added_by_the_sweeps_equal_a_launch_of_their_own(shape, L):
    """Up to 1024 sources are added by the pressure sweep; one more source, of
    weight zero, makes the same sources take a launch of their own."""
    rng = np.random.default_rng(L)
    prob = W.random_medium(shape, L, 2, seed=4, nb=3, ntr=2)
    idx = rng.choice(prob.npts, 1025, replace=False).astype(np.int64)
    prob.signals = (1e4 * rng.standard_normal((2, 5))).astype(np.float32)    # ends within the run
    prob.rcv_idx = idx[:7]
    got = []
    for n in (1024, 1025):
        prob.src_idx, prob.src_sig = idx[:n], (np.arange(n) % 2).astype(np.int32)
        prob.src_w = np.append(rng.uniform(0.5, 1.0, 1024) if not got else got[0][2][:1024],
                               [0.0])[:n].astype(np.float32)
        dom = fw2.from_problem(prob, device="cuda:0", cap_steps=7)
        dom.step(7)
        got.append((dom.read_fields(fw2.FIELD_ALL), dom.trace.cpu().numpy(), prob.src_w))
        dom.destroy_domain()
    for k in got[0][0]:
        assert np.array_equal(got[0][0][k], got[1][0][k]), k
    assert np.array_equal(got[0][1], got[1][1]) and np.any(got[0][1])
