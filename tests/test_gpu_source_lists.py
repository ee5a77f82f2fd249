"""Sources added by the tiles and by a launch of their own give the same bits:
in a batch, in the one-launch step and in the tiled reverse step, at 4096
sources and at 4 Mi pairs of a tile and a source.  Sources of weight zero move
a run across a limit without changing what it computes."""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu


def _problem(shape, L, n_src, n_zero=0, seed=0, n_t=12):
    """n_src sources of any weight, then n_zero of weight zero."""
    rng = np.random.default_rng(seed)
    prob = W.homogeneous(shape, L=L, nb=(6, 6))
    prob.src_idx = rng.choice(prob.npts, n_src + n_zero, replace=False).astype(np.int64)
    prob.src_sig = rng.integers(0, 2, n_src + n_zero).astype(np.int32)
    prob.src_w = np.where(np.arange(n_src + n_zero) < n_src, rng.uniform(0.5, 1.0, n_src + n_zero), 0.0).astype(np.float32)
    prob.signals = (1e4 * np.random.default_rng(seed + 1).standard_normal((2, n_t))).astype(np.float32)
    prob.rcv_idx = np.random.default_rng(seed + 2).choice(prob.npts, 9, replace=False).astype(np.int64)
    return prob


def _trim(prob, n):
    """The same run without the sources past the first n."""
    q = W.Problem(**{k: getattr(prob, k) for k in prob.__dataclass_fields__})
    q.src_idx, q.src_sig, q.src_w = prob.src_idx[:n], prob.src_sig[:n], prob.src_w[:n]
    return q


def _result(dom):
    from paper_2106_11476_amd import fw2
    return dict(dom.read_fields(fw2.FIELD_ALL), trace=dom.trace.cpu().numpy())


def _equal(a, b, what):
    for k in a:
        assert np.array_equal(a[k], b[k]), (what, k)


def _solo(prob, n):
    from paper_2106_11476_amd import fw2
    dom = fw2.from_problem(prob, device="cuda:0", cap_steps=n)
    dom.step(n)
    out = _result(dom)
    dom.destroy_domain()
    return out


def test_batches_at_the_source_limits_equal_solo_runs():
    """A domain of few sources beside one of 4096, then of 4097 (a launch of
    their own), then of few again: the captured step follows each change."""
    torch = _torch()
    from paper_2106_11476_amd import fw2
    stream = torch.cuda.Stream()
    n = 70                                       # two captured loops of 32 steps and 6 by themselves
    few = _problem((130, 70), 2, 5, seed=3)
    few_ref = _solo(few, n)
    batch = fw2.Batch(max_domains=4, stream=stream)
    for n_src in (4096, 4097, 17, 4097):
        _say("batch with", n_src, "sources")
        many = _problem((140, 90), 3, n_src, seed=n_src)
        probs = [few, many]
        doms = [fw2.from_problem(p, device="cuda:0", stream=stream, cap_steps=n) for p in probs]
        batch.set_domains(doms, [n, n])
        batch.step(n)
        stream.synchronize()
        _equal(_result(doms[0]), few_ref, n_src)
        _equal(_result(doms[1]), _solo(many, n), n_src)
        batch.set_domains([], [])
        for d in doms:
            d.destroy_domain()
    batch.destroy()


@pytest.mark.parametrize("n_zero", [0, 40])
def test_batch_at_the_pair_limit(n_zero):
    """1024 x 768 and 1024 x 256: 2048 tiles of 64 x 8 together, 2048 sources
    in each make 4 Mi pairs."""
    torch = _torch()
    from paper_2106_11476_amd import fw2
    _say("batch pairs, zero-weight sources", n_zero)
    stream = torch.cuda.Stream()
    probs = [_problem((1024, 768), 1, 2048, n_zero, seed=5), _problem((1024, 256), 2, 2048, 0, seed=6)]
    doms = [fw2.from_problem(p, device="cuda:0", stream=stream, cap_steps=9) for p in probs]
    batch = fw2.Batch(max_domains=2, stream=stream)
    batch.set_domains(doms, [9, 9])
    batch.step(9)
    stream.synchronize()
    for d, p in zip(doms, probs):
        _equal(_result(d), _solo(_trim(p, 2048), 9), n_zero)
    batch.destroy()
    for d in doms:
        d.destroy_domain()


def test_one_launch_step_at_the_pair_limit():
    """1500 x 1500: 2256 tiles of 64 x 16; 1859 sources are the last that the
    one launch adds."""
    _torch()
    _say("one-launch pairs")
    prob = _problem((1500, 1500), 1, 1859, 1, seed=8)
    _equal(_solo(prob, 7), _solo(_trim(prob, 1859), 7), "1860 / 1859")


def test_reverse_steps_at_the_pair_limit():
    """1040 x 1030: 17 x 129 tiles of 64 x 8; the gradient with 1900 sources
    in the tiles, and with 100 more of weight zero by a launch."""
    torch = _torch()
    from paper_2106_11476_amd import adjoint
    prob = _problem((1040, 1030), 1, 1900, 100, seed=9)
    prob.fd_r, prob.pml_cp = float(prob.c.max()) * prob.dt / prob.h, float(prob.c.max())
    _say("reverse pairs")
    grads = []
    for p in (prob, _trim(prob, 1900)):
        c = torch.tensor(np.asarray(p.c, np.float64), requires_grad=True)
        obs = torch.zeros((10, p.rcv_idx.size), device="cuda:0")
        adjoint.misfit(c, obs, p, 10, checkpoint_every=5).backward()
        grads.append(c.grad.numpy())
    assert np.abs(grads[0]).max() > 0 and np.array_equal(grads[0], grads[1])
