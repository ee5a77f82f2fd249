"""Performance cases of the library: what its users have it do, through the
public entry points of paper_2106_11476_amd.

A case is a dict of plain values; its "kind" is the way the library is used:

  poll        one time step and the pressure field read back after it (a
              program coupled to the solver, or one that draws every step)
  event       a transmit event: a stored state loaded, n steps with sources
              and receivers, then the traces and a snapshot of the fields
  batch       many small 2D domains advanced together (serving)
  slabs       a 3D grid split along z, stepped with halo exchange
  gradient    the trace misfit and its sound-speed gradient (autograd)
  reverse     reverse steps over stored forward states, then the gradient
  checkpoint  all fields written, a step, all fields read (resume and save)

prepare() makes the inputs from the seed and builds what such a program keeps
(domains, state blocks); run() is one pass; work() is what the pass cannot do
without; exact() is the same pass in 64 bits in plain torch, written from the
method's formulas (staggered (8,4) stencil, memory variables, two-stage C-PML).
"""
import math
from dataclasses import dataclass, field

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

from paper_2106_11476_amd import adjoint, fw2, slab

DEV = "cuda" if torch.cuda.is_available() else "cpu"
FIELDS = {"p": fw2.FIELD_P, "pv": fw2.FIELD_P | fw2.FIELD_V, "all": fw2.FIELD_ALL}


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def _event(name, shape, L, n, **kw):
    c = {"name": name, "kind": "event", "nx": shape[0], "ny": shape[1], "nz": shape[2] if len(shape) == 3 else 0,
         "L": L, "labels": 9, "nb": 48, "n": n, "src": 64, "rcv": 64, "printed": False, "local": False,
         "custom": False, "read": "pv"}
    c.update(kw)
    return c


def listed():
    return [
        # The smallest call: one step of a small water tank, its pressure read back.
        {"name": "poll_2d_128", "kind": "poll", "nx": 128, "ny": 128, "L": 2, "nb": 16, "src": 16},
        # The plain 2D workload's grid: too small to fill the GPU, bound by launches.
        _event("event_2d_480", (480, 480), 2, 100, labels=1, src=384, read="all"),
        # A served 2D request of the smallest served size.
        _event("event_2d_1024_L3", (1024, 1024), 3, 64, src=640, rcv=64),
        # The heterogeneous abdominal grid with its 128-element array: ordinary production in 2D.
        _event("event_2d_4096x2048_L4", (4096, 2048), 4, 32, src=1280, rcv=128),
        # Ragged sizes with the options: 8 mechanisms, printed recursion, per-point weights.
        _event("event_2d_1237x893_L8", (1237, 893), 8, 32, nb=37, printed=True, local=True),
        # A transcranial cube far larger than the caches (the headline's kernels).
        _event("event_3d_512", (512, 512, 512), 2, 6, labels=2, src=1024, read="p"),
        # A ragged 3D grid with the custom nonlinear form and the printed recursion.
        _event("event_3d_203x149x177", (203, 149, 177), 3, 16, nb=21, printed=True, custom=True),
        # Three slabs of a grid split along z, the decomposition's one-GPU part.
        {"name": "slabs_3d_256x256x192", "kind": "slabs", "nx": 256, "ny": 256, "nz": 192, "L": 2, "slabs": 3, "n": 8},
        # Serving: requests too small to fill the GPU, stepped together to completion.
        {"name": "batch_2d_32", "kind": "batch", "count": 32, "lo": 128, "hi": 384, "n": 64},
        # Full waveform inversion: misfit and gradient of one shot through autograd.
        {"name": "gradient_2d_384", "kind": "gradient", "nx": 384, "ny": 384, "L": 2, "n": 192, "rcv": 128},
        # The reverse half of one checkpoint segment at the inversion workload's size.
        {"name": "reverse_2d_1536", "kind": "reverse", "nx": 1536, "ny": 1536, "nz": 0, "L": 2, "n": 32, "rcv": 256},
        # Checkpoint and resume of a 3D run.
        {"name": "checkpoint_3d_160", "kind": "checkpoint", "nx": 160, "ny": 160, "nz": 160, "L": 2},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["poll", "event", "event", "event3", "event3", "slabs", "batch", "gradient", "reverse",
                       "checkpoint"])
    L = rng.choice([1, 2, 2, 3, 4, 4, 6])
    if kind == "poll":
        return {"kind": "poll", "nx": _log(rng, 96, 700), "ny": _log(rng, 96, 700), "L": L,
                "nb": rng.randint(8, 24), "src": rng.randint(1, 48)}
    if kind == "event":
        shape = (_log(rng, 96, 4096), _log(rng, 96, 2048))
        n = max(4, min(200, int(2.5e8 / (shape[0] * shape[1]))))
        nb = rng.randint(8, min(48, min(shape) // 4))
    elif kind == "event3":
        shape = tuple(_log(rng, 40, 400) for _ in range(3))
        n = max(2, min(64, int(2.5e8 / (shape[0] * shape[1] * shape[2]))))
        nb = rng.randint(4, min(32, min(shape) // 4))
    if kind in ("event", "event3"):
        c = _event("", shape, L, n, labels=rng.choice([1, 2, 9]), nb=nb, src=rng.randint(1, 512),
                   rcv=rng.randint(1, 128), printed=rng.random() < 0.3, local=rng.random() < 0.3,
                   custom=rng.random() < 0.3, read=rng.choice(["p", "pv", "all"]))
        del c["name"]
        return c
    if kind == "slabs":
        return {"kind": "slabs", "nx": _log(rng, 64, 320), "ny": _log(rng, 64, 320), "nz": rng.randint(64, 200),
                "L": rng.choice([2, 3]), "slabs": rng.randint(2, 4), "n": rng.randint(2, 8)}
    if kind == "batch":
        lo = _log(rng, 96, 200)
        return {"kind": "batch", "count": rng.randint(4, 48), "lo": lo, "hi": rng.randint(lo + 1, 400),
                "n": rng.randint(16, 64)}
    if kind == "gradient":
        return {"kind": "gradient", "nx": _log(rng, 128, 512), "ny": _log(rng, 128, 512), "L": rng.choice([1, 2, 3]),
                "n": rng.randint(64, 192), "rcv": rng.randint(8, 128)}
    if kind == "reverse":
        if rng.random() < 0.3:
            return {"kind": "reverse", "nx": _log(rng, 48, 128), "ny": _log(rng, 48, 128), "nz": _log(rng, 48, 128),
                    "L": rng.choice([1, 2]), "n": rng.randint(4, 16), "rcv": rng.randint(8, 128)}
        return {"kind": "reverse", "nx": _log(rng, 256, 1600), "ny": _log(rng, 256, 1600), "nz": 0,
                "L": rng.choice([1, 2, 3]), "n": rng.randint(8, 32), "rcv": rng.randint(8, 256)}
    return {"kind": "checkpoint", "nx": _log(rng, 48, 200), "ny": _log(rng, 48, 200), "nz": _log(rng, 48, 200),
            "L": rng.choice([1, 2, 3])}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

@dataclass
class Simulation:
    """The fields fw2.Domain reads (grids are [nz][ny][nx], x fastest)."""
    shape: tuple
    h: float
    dt: float
    n_relax: int
    c: object
    rho: object
    beta: object
    relax_table: object
    label: object = None
    bound_cells: tuple = (0, 0, 0)
    trans_cells: tuple = (0, 0, 0)
    pml_Rc: float = 1e-3
    pml_npoly: int = 2
    pml_cp: float = 0.0
    fd_r: float = 0.0
    relax_scheme: int = 1
    stencil_mode: int = 0
    nonlinear_form: int = 0
    nl_A: float = 1.0
    nl_B0: float = 1.0
    nl_B1: float = -2.0
    src_idx: object = field(default_factory=lambda: np.zeros(0, np.int64))
    src_sig: object = field(default_factory=lambda: np.zeros(0, np.int32))
    src_w: object = field(default_factory=lambda: np.zeros(0, np.float32))
    signals: object = field(default_factory=lambda: np.zeros((1, 1), np.float32))
    rcv_idx: object = field(default_factory=lambda: np.zeros(0, np.int64))
    n_steps: int = 0
    name: str = ""


def _relax_row(L, strength):
    """Relaxation tuple of one tissue: the paper's Table 2 for L = 2, else
    mechanisms spread over its range of relaxation rates."""
    if L == 2:
        d1, d2 = [9.82e5, 3.26e6], [4.40e4, 1.68e5]
        a1, a2 = [2.83e8, 3.54e9], [8.35e6, 5.10e7]
        k1, k2 = 0.835, 1.19
    else:
        a2 = list(np.logspace(6.7, 8.7, L))
        a1 = list(np.logspace(7.3, 9.4, L))
        d1, d2 = [0.004 / L * a for a in a1], [0.004 / L * a for a in a2]
        k1, k2 = 0.9, 1.1
    return [k1, k2] + [strength * d for d in d1] + [strength * d for d in d2] + a1 + a2


def _pulse(n, period, amp):
    """Gaussian-modulated sinusoid centred in n samples."""
    t = np.arange(n) + 0.5 - n / 2
    return amp * np.sin(2 * np.pi * t / period) * np.exp(-0.5 * (t / (0.75 * period)) ** 2)


def _simulation(shape, L, labels, nb, n, src, rcv, seed, printed=False, local=False, custom=False, fixed=False):
    """A layered tissue medium with scatterers (2D) or a background with a
    bone-like shell (3D, two labels); a transducer row of sources and a row of
    receivers near the top; 12 points per wavelength at 3 MHz, CFL 0.4."""
    nd = len(shape)
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    grid = tuple(shape[::-1])
    depth = torch.arange(grid[0], device=DEV, dtype=torch.float32).reshape((-1,) + (1,) * (nd - 1))
    lateral = [torch.arange(n_, device=DEV, dtype=torch.float32).reshape((1,) * (k + 1) + (-1,) + (1,) * (nd - 2 - k))
               for k, n_ in enumerate(grid[1:])]
    wave = sum(0.02 * grid[0] * torch.sin(2 * math.pi * (rng.uniform(1, 3) * x / x.numel() + rng.uniform()))
               for x in lateral)
    layer = torch.zeros(grid, dtype=torch.uint8, device=DEV)
    if nd == 3 and labels == 2:
        top = 0.4 * grid[0] + wave
        layer |= ((depth >= top) & (depth < top + 6)).to(torch.uint8)
        cs, rhos, betas = [1540.0, 2800.0], [1040.0, 1900.0], [4.0, 4.0]
    else:
        for q in np.sort(rng.uniform(0.1, 0.9, max(labels - 1, 0))) * grid[0]:
            layer += (depth >= q + wave).to(torch.uint8)
        m = max(labels, 1)
        cs, rhos, betas = rng.uniform(1450, 1620, m), rng.uniform(950, 1120, m), rng.uniform(3.5, 5.5, m)
    val = {}
    for name, v in (("c", cs), ("rho", rhos), ("beta", betas)):
        val[name] = torch.tensor(np.asarray(v), dtype=torch.float32, device=DEV)[layer.int()]
    npts = layer.numel()
    at = torch.randint(0, npts, (min(100000, npts // 50 + 1),), generator=gen, device=DEV).unique()
    val["c"].view(-1)[at] *= 1 + 0.02 * torch.randn(at.numel(), generator=gen, device=DEV).clamp(-3, 3)
    h = 1540.0 / (12 * 3e6)
    cmax = float(val["c"].max())
    dt = 0.4 * h / cmax
    s = Simulation(shape=tuple(shape), h=h, dt=dt, n_relax=L,
                   c=val["c"].cpu().numpy(), rho=val["rho"].cpu().numpy(), beta=val["beta"].cpu().numpy(),
                   relax_table=np.array([_relax_row(L, rng.uniform(0.8, 1.2)) for _ in range(max(labels, 1))]),
                   label=layer.cpu().numpy() if labels > 1 else None,
                   bound_cells=(nb,) * nd, trans_cells=(nb * 3 // 4,) * nd,
                   relax_scheme=0 if printed else 1, stencil_mode=1 if local else 0, n_steps=n)
    if fixed:                                       # constants that do not follow c
        s.fd_r, s.pml_cp = cmax * dt / h, cmax
    if custom:                                      # the Westervelt coefficient
        s.nonlinear_form, s.nl_A, s.nl_B0, s.nl_B1 = 1, 0.0, 0.0, -2.0
    row = min(nb + 8, grid[0] - 1)
    nx, plane = shape[0], int(np.prod(shape[:-1]))
    start = row * plane + (nx * (shape[1] // 2) if nd == 3 else 0)   # first point of the transducer's row or plane
    room = plane if nd == 2 else plane - nx * (shape[1] // 2)
    lead = nb if nd == 2 else 0
    if src:
        k = min(src, max(room - 2 * lead, 1))
        s.src_idx = (start + lead + np.arange(k)).astype(np.int64)
        s.src_sig = (np.arange(k) * min(k, 8) // k).astype(np.int32)
        s.src_w = rng.uniform(0.5, 1.0, k).astype(np.float32)
        s.signals = np.stack([_pulse(n, 30.0, 1e5 * rng.uniform(0.5, 1.0)) for _ in range(min(k, 8))]).astype(np.float32)
    if rcv:
        k = min(rcv, max(nx - 2 * nb, 1))
        at = nb + (np.arange(k) * max(nx - 2 * nb, 1)) // k
        s.rcv_idx = (min(row + 4, grid[0] - 1) * plane + start - row * plane + at).astype(np.int64)
    return s


def _state(sim, seed):
    """Packed random state (p, v, psi1, psi2) at acoustic magnitudes; velocity
    samples past the grid are zero."""
    gen = torch.Generator(device=DEV).manual_seed(seed + 1000003)
    nd, L, grid = len(sim.shape), sim.n_relax, tuple(sim.shape[::-1])
    npts = int(np.prod(grid))
    buf = torch.empty((1 + nd + 2 * nd * L, npts), dtype=torch.float32, device=DEV)
    for k in range(buf.shape[0]):
        scale = 1e5 if k == 0 else 0.067 if k <= nd else 1e3 if k <= nd + nd * L else 6.7
        torch.randn(npts, generator=gen, device=DEV, out=buf[k])
        buf[k] *= scale
        a = k - 1 if 1 <= k <= nd else (k - 1 - nd) // L if nd < k <= nd + nd * L else -1
        if a >= 0:                                  # v_a and psi1[a]: the last sample along a
            buf[k].view(grid).narrow(nd - 1 - a, grid[nd - 1 - a] - 1, 1).zero_()
    return buf.view(-1)


def _slab_state(case, sim, seed):
    """_state with the last v_z and psi1[z] plane of every slab zero (a field
    write leaves a domain's last sample along each axis at zero)."""
    nz, L = case["nz"], case["L"]
    bounds = [nz * k // case["slabs"] for k in range(case["slabs"] + 1)]
    views = _state(sim, seed).view(-1, nz, case["ny"], case["nx"])
    for b in bounds[1:]:
        views[3, b - 1].zero_()
        views[4 + 2 * L:4 + 3 * L, b - 1].zero_()
    return bounds, views


def _shape(case):
    return (case["nx"], case["ny"]) + ((case["nz"],) if case.get("nz") else ())


def _case_simulation(case, seed):
    k = case["kind"]
    if k == "poll":
        return _simulation(_shape(case), case["L"], 1, case["nb"], 200, case["src"], 0, seed)
    if k == "event":
        return _simulation(_shape(case), case["L"], case["labels"], case["nb"], case["n"], case["src"], case["rcv"],
                           seed, case["printed"], case["local"], case["custom"])
    if k == "slabs":
        return _simulation(_shape(case), case["L"], 2, 16, case["n"], 64, 32, seed, fixed=True)
    if k in ("gradient", "reverse"):
        nb = 8 if case.get("nz") else 24
        return _simulation(_shape(case), case["L"], 5, nb, case["n"], 1, case["rcv"], seed, fixed=True)
    return _simulation(_shape(case), case["L"], 2, 8, 16, 8, 0, seed)       # checkpoint


def _batch_simulations(case, seed):
    rng = np.random.default_rng(seed)
    out = []
    # the mix of sizes and options belongs to the case, the inputs to the seed
    mix = np.random.default_rng(case["count"] * 1000003 + case["lo"] * 1009 + case["hi"])
    for _ in range(case["count"]):
        shape = tuple(int(v) for v in mix.integers(case["lo"], case["hi"] + 1, 2))
        L, printed = int(mix.integers(2, 5)), bool(mix.integers(0, 2))
        out.append(_simulation(shape, L, 4, 20, case["n"], 32, 16, int(rng.integers(1 << 30)), printed))
    return out


def _observed(case, seed):
    """Smooth observed traces [n, rcv] of the misfit (or a residual)."""
    rng = np.random.default_rng(seed + 7)
    sim = _case_simulation(case, seed)
    k = len(sim.rcv_idx)
    t = np.arange(case["n"])[:, None]
    ph, fr = rng.uniform(0, 2 * np.pi, (3, 1, k)), rng.uniform(0.02, 0.06, (3, 1, k))
    return sim, (3e3 * sum(np.sin(2 * np.pi * fr[q] * t + ph[q]) for q in range(3))).astype(np.float32)


# ---------------------------------------------------------------------------
# One pass through the library
# ---------------------------------------------------------------------------

def _domain(sim, state=None, device_maps=False):
    dom = fw2.Domain(sim, device=DEV, device_maps=device_maps)
    if len(sim.src_idx):
        dom.add_source(sim.src_idx, sim.src_sig, sim.src_w, sim.signals)
    if len(sim.rcv_idx):
        dom.add_receivers(sim.rcv_idx, sim.n_steps)
    if state is not None:
        dom.write_fields_device(state)
    return dom


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        sims = _batch_simulations(case, seed)
        doms, starts = [], []
        for k, sim in enumerate(sims):
            dom = _domain(sim, _state(sim, seed + k))
            starts.append(dom.new_state_buffer())
            dom.save_state(starts[-1])
            doms.append(dom)
        batch = fw2.Batch(max_domains=len(doms), device=DEV, stream=torch.cuda.current_stream())
        return {"case": case, "doms": doms, "starts": starts, "batch": batch}
    if kind == "gradient":
        sim, obs = _observed(case, seed)
        return {"case": case, "sim": sim, "obs": torch.as_tensor(obs, device=DEV),
                "c": torch.as_tensor(sim.c, device=DEV).requires_grad_(True)}
    if kind == "reverse":
        sim, res = _observed(case, seed)
        dom = _domain(sim, _state(sim, seed))
        seg = dom.new_state_buffer(case["n"])
        dom.save_state(seg[0])
        dom.step_into(case["n"] - 1, seg[0], seg[1:])
        return {"case": case, "dom": dom, "seg": seg, "res": torch.as_tensor(res, device=DEV)}
    sim = _case_simulation(case, seed)
    if kind == "slabs":
        bounds, views = _slab_state(case, sim, seed)
        whole = slab.SlabSet(sim, bounds, device=DEV)
        for k, dom in enumerate(whole.domains):
            dom.write_fields_device(views[:, bounds[k]:bounds[k + 1]].contiguous().view(-1))
        whole.exchange(fw2.HALO_V)
        starts = []
        for dom in whole.domains:
            starts.append(dom.new_state_buffer())
            dom.save_state(starts[-1])
        return {"case": case, "set": whole, "starts": starts}
    state = _state(sim, seed)
    dom = _domain(sim, state, device_maps=len(sim.shape) == 3)
    out = {"case": case, "dom": dom}
    if kind == "event":
        out["start"] = dom.new_state_buffer()
        dom.save_state(out["start"])
    elif kind == "checkpoint":
        out["state"] = state
    return out


def _fields(dom, mask):
    return dom.field_views(dom.read_fields_device(mask), mask)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "poll":
        dom = state["dom"]
        dom.step(1)
        return _fields(dom, fw2.FIELD_P)
    if kind == "event":
        dom = state["dom"]
        dom.load_state(state["start"], 0)
        dom.step(case["n"])
        return {"trace": dom.trace, **_fields(dom, FIELDS[case["read"]])}
    if kind == "batch":
        doms, batch = state["doms"], state["batch"]
        for dom, start in zip(doms, state["starts"]):
            dom.load_state(start, 0)
        batch.set_domains(doms, [case["n"]] * len(doms))
        batch.step(case["n"])
        batch.set_domains([], [])
        return [d.trace for d in doms[:16]] + [_fields(d, fw2.FIELD_P) for d in doms]
    if kind == "slabs":
        s = state["set"]
        for dom, start in zip(s.domains, state["starts"]):
            dom.load_state(start, 0)
        s.step(case["n"])
        return [_fields(d, FIELDS["pv"]) for d in s.domains]
    if kind == "gradient":
        c = state["c"]
        c.grad = None
        loss = adjoint.misfit(c, state["obs"], state["sim"], case["n"])
        loss.backward()
        return {"misfit": loss.detach().to(torch.float32), "gradient": c.grad}
    if kind == "reverse":
        dom, seg, res = state["dom"], state["seg"], state["res"]
        dom.adjoint_begin()
        for k in reversed(range(case["n"])):
            dom.adjoint_step(seg[k], k, res[k], prev=seg[k - 1] if k else None)
        return dom.adjoint_gradient()
    dom = state["dom"]
    dom.write_fields_device(state["state"])
    dom.set_current_step(0)
    dom.step(1)
    return _fields(dom, fw2.FIELD_ALL)


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

def _point_bytes(nd, L, labels):
    """State and medium per point: bytes of the state, of the three medium
    values with the label."""
    return 4 * (1 + nd + 2 * nd * L), 12 + (1 if labels > 1 else 0)


def _point_flops(nd, L, local=False):
    """One step of one point: per axis and phase the stencil (4 pairs and the
    cross pairs), the memory variables (two fused multiply-adds each) and the
    update; per-point weights add four cubics."""
    return 2 * nd * (11 + 4 * (nd - 1) + 4 * L + 8) + (2 * nd * 26 if local else 0)


def work(case):
    """Steps run in turn and a state of this size does not stay on the chip,
    so every step reads and writes the state once and reads the medium once;
    a reverse step reads the forward state and the medium and reads and writes
    the adjoint state and the gradient."""
    kind = case["kind"]
    if kind == "batch":
        b = f = 0
        mix = np.random.default_rng(case["count"] * 1000003 + case["lo"] * 1009 + case["hi"])
        for _ in range(case["count"]):
            npts = int(np.prod(mix.integers(case["lo"], case["hi"] + 1, 2)))
            L, _ = int(mix.integers(2, 5)), mix.integers(0, 2)
            s, m = _point_bytes(2, L, 4)
            b += npts * case["n"] * (2 * s + m) + npts * (2 * s + 8)
            f += npts * case["n"] * _point_flops(2, L)
        return {"bytes": b, "flops": f}
    shape = _shape(case)
    nd, npts, L = len(shape), int(np.prod(shape)), case["L"]
    labels = case.get("labels", {"poll": 1, "gradient": 5, "reverse": 5}.get(kind, 2))
    s, m = _point_bytes(nd, L, labels)
    step, flops = 2 * s + m, _point_flops(nd, L, case.get("local", False))
    back = 3 * s + m + 8
    if kind == "poll":
        return {"bytes": npts * (step + 8), "flops": npts * flops}
    if kind == "event":
        out = {"p": 8, "pv": 8 * (1 + nd), "all": 2 * s}[case["read"]]
        return {"bytes": npts * (case["n"] * step + 2 * s + out), "flops": npts * case["n"] * flops}
    if kind == "slabs":
        return {"bytes": npts * (case["n"] * step + 2 * s + 8 * (1 + nd)), "flops": npts * case["n"] * flops}
    if kind == "gradient":
        return {"bytes": npts * case["n"] * (2 * step + back), "flops": npts * case["n"] * 4 * flops}
    if kind == "reverse":
        return {"bytes": npts * case["n"] * back, "flops": npts * case["n"] * 2 * flops}
    return {"bytes": npts * (step + 4 * s), "flops": npts * flops}


# ---------------------------------------------------------------------------
# The same pass in 64 bits
# ---------------------------------------------------------------------------

def _weights(r2, nd):
    """Stencil weights of the (8,4) operator at Courant number squared r2 (a
    number or a tensor): sum_j c_j (2j-1)^(2k-1) = r2^(k-1), g11 = r2 / 24."""
    A = np.array([[(2.0 * j - 1) ** (2 * k - 1) for j in range(1, 5)] for k in range(1, 5)])
    inv = np.linalg.inv(A)
    g = [sum(float(inv[j, k]) * r2 ** k for k in range(4)) for j in range(4)]
    g11 = r2 / 24.0
    g[0] = g[0] - 2.0 * (nd - 1) * g11
    return g, g11


class _Exact:
    """Coefficients of one simulation in 64 bits; c may carry a gradient."""

    def __init__(self, sim, c=None):
        self.sim, self.nd, self.L = sim, len(sim.shape), sim.n_relax
        self.grid = tuple(sim.shape[::-1])
        f64 = dict(dtype=torch.float64, device=DEV)
        self.c = torch.as_tensor(sim.c, **f64) if c is None else c
        self.rho = torch.as_tensor(sim.rho, **f64)
        beta = torch.as_tensor(sim.beta, **f64)
        A, B0, B1 = (sim.nl_A, sim.nl_B0, sim.nl_B1) if sim.nonlinear_form else (1.0, 1.0, -2.0)
        self.A = A
        self.B = B0 + B1 * beta
        self.label = None if sim.label is None else torch.as_tensor(sim.label, device=DEV)
        cmax = float(np.max(sim.c))
        self.cp = sim.pml_cp if sim.pml_cp > 0 else cmax
        r = sim.fd_r if sim.fd_r > 0 else cmax * sim.dt / sim.h
        self.g = _weights(r * r, self.nd)
        self.tables = {}

    def kappa(self):
        return 1.0 / (self.rho * self.c * self.c)

    def table(self, nabla, a):
        """w, (b, c) per mechanism at every coordinate along a and label:
        [n_a, n_labels] arrays of the memory recursion."""
        if (nabla, a) in self.tables:
            return self.tables[nabla, a]
        sim, L, n, nb, ntr = self.sim, self.L, self.sim.shape[a], self.sim.bound_cells[a], self.sim.trans_cells[a]
        x = np.arange(n) + (0.5 if nabla == 1 else 0.0)
        s = np.clip(np.maximum(nb - x, x - (n - 1 - nb)), 0.0, nb)[:, None]
        rows, dt = np.asarray(sim.relax_table), sim.dt
        kap = rows[:, nabla - 1][None, :]
        w, bs, cs = 1.0 / kap + 0 * s, [], []
        for nu in range(L):
            d0 = rows[:, 2 + (nabla - 1) * L + nu][None, :]
            a0 = rows[:, 2 + (nabla + 1) * L + nu][None, :]
            if nb == 0:
                d, al = d0 + 0 * s, a0 + 0 * s
            elif nu == 0:
                target = -(sim.pml_npoly + 1) * self.cp * math.log(sim.pml_Rc) / (2 * nb * sim.h)
                d = (target - d0) * (s / nb) ** sim.pml_npoly + d0
                al = a0 * (1 - s / nb)
            else:
                ramp = 0.5 * (1 - np.cos(np.pi * np.minimum(s, ntr) / ntr)) if ntr > 0 else 0 * s
                d, al = d0 * (1 - ramp), a0 * (1 - ramp)
            lam = d / kap + al
            b = np.exp(-lam * dt)
            safe = np.where(d == 0, 1.0, lam)
            za = np.where(d == 0, 0.0, d / (kap * kap * safe) * np.expm1(-safe * dt))
            e1 = np.where(d == 0, 0.0, -d / kap ** 2 * (-np.expm1(-safe * dt) - safe * dt * np.exp(-safe * dt))
                          / (safe * safe * dt))
            e0 = za - e1
            bs.append(b)
            if sim.relax_scheme:
                w = w + e0
                cs.append(e1 + b * e0)
            else:
                cs.append(za)
        out = (w, bs, cs)
        self.tables[nabla, a] = out
        return out

    def at(self, tab, a):
        """A [n_a, n_labels] array at every point."""
        t = torch.as_tensor(tab, dtype=torch.float64, device=DEV)
        shape = [1] * self.nd
        shape[self.nd - 1 - a] = -1
        if self.label is None:
            return t[:, 0].reshape(shape)
        at = torch.arange(t.shape[0], device=DEV).reshape(shape) * t.shape[1] + self.label
        return t.reshape(-1)[at]

    def take(self, f, off):
        """The zero-padded field f at x + off (off per physical axis)."""
        for a in range(self.nd):
            f = f.narrow(self.nd - 1 - a, 4 + off[a], self.sim.shape[a])
        return f

    def derivative(self, f, a, nabla, g):
        """D^+ (nabla 1) or D^- (nabla 2) of f along a, over h."""
        fp = torch.nn.functional.pad(f, (4, 4) * self.nd)
        lead = 1 if nabla == 1 else 0

        def e(k, b=None, sb=0):
            o = [0, 0, 0]
            o[a] += k
            if b is not None:
                o[b] += sb
            return self.take(fp, o)

        w, g11 = g
        D = 0.0
        for m in range(4):
            D = D + w[m] * (e(m + lead) - e(lead - 1 - m))
        cross = 0.0
        for b in range(self.nd):
            if b != a:
                for sb in (1, -1):
                    cross = cross + (e(lead, b, sb) - e(lead - 1, b, sb))
        return (D + g11 * cross) / self.sim.h

    def ahead(self, f, a):
        """f at the next point along a (the last value repeated)."""
        d = self.nd - 1 - a
        n = f.shape[d]
        return torch.cat([f.narrow(d, 1, n - 1), f.narrow(d, n - 1, 1)], d) if n > 1 else f

    def memory(self, nabla, a, D, psi):
        w, bs, cs = self.table(nabla, a)
        S, new = self.at(w, a) * D, []
        for nu in range(self.L):
            m = self.at(bs[nu], a) * psi[nu] + self.at(cs[nu], a) * D
            S = S + (psi[nu] if self.sim.relax_scheme else m)
            new.append(m)
        return S, new

    def step(self, state, k):
        """One step from state = (p, v..., psi1..., psi2...); returns the next
        state and the pressures at the receivers."""
        sim, nd, L = self.sim, self.nd, self.L
        p, v = state[0], list(state[1:1 + nd])
        psi1 = [list(state[1 + nd + a * L:1 + nd + (a + 1) * L]) for a in range(nd)]
        psi2 = [list(state[1 + nd + (nd + a) * L:1 + nd + (nd + a + 1) * L]) for a in range(nd)]
        kap = self.kappa()
        r2 = (self.c * (sim.dt / sim.h)) ** 2 if sim.stencil_mode else None
        S = 0.0
        g = _weights(r2, nd) if sim.stencil_mode else self.g
        for a in range(nd):
            Sa, psi2[a] = self.memory(2, a, self.derivative(v[a], a, 2, g), psi2[a])
            S = S + Sa
        p = p - sim.dt * S / (kap * (1 + kap * self.B * p))
        if len(sim.src_idx) and k < sim.signals.shape[1]:
            amount = torch.as_tensor(sim.src_w, dtype=torch.float64, device=DEV) * torch.as_tensor(
                sim.signals[sim.src_sig, k], dtype=torch.float64, device=DEV)
            p = p.reshape(-1).index_add(0, torch.as_tensor(sim.src_idx, device=DEV), amount).reshape(self.grid)
        seen = p.reshape(-1)[torch.as_tensor(sim.rcv_idx, device=DEV)]
        for a in range(nd):
            g = _weights(0.5 * (r2 + self.ahead(r2, a)), nd) if sim.stencil_mode else self.g
            Sa, new = self.memory(1, a, self.derivative(p, a, 1, g), psi1[a])
            pbar, ra = 0.5 * (p + self.ahead(p, a)), 0.5 * (self.rho + self.ahead(self.rho, a))
            ka = 0.5 * (kap + self.ahead(kap, a))
            inside = torch.ones(self.grid[nd - 1 - a], dtype=torch.float64, device=DEV)
            inside[-1] = 0.0                        # the sample past the grid stays zero
            shape = [1] * nd
            shape[nd - 1 - a] = -1
            inside = inside.reshape(shape)
            v[a] = (v[a] - sim.dt * Sa / (ra * (1 + self.A * ka * pbar))) * inside
            psi1[a] = [m * inside for m in new]
        return tuple([p] + v + sum(psi1, []) + sum(psi2, [])), seen

    def split(self, packed):
        s = packed.double().view((-1,) + self.grid)
        return tuple(s[k] for k in range(s.shape[0]))

    def packed(self, state, mask):
        nd, L = self.nd, self.L
        out = {}
        for name, bit, lo, hi, lead in (("p", fw2.FIELD_P, 0, 1, ()), ("v", fw2.FIELD_V, 1, 1 + nd, (nd,)),
                                        ("psi1", fw2.FIELD_PSI1, 1 + nd, 1 + nd + nd * L, (nd, L)),
                                        ("psi2", fw2.FIELD_PSI2, 1 + nd + nd * L, 1 + nd + 2 * nd * L, (nd, L))):
            if mask & bit:
                out[name] = torch.stack(state[lo:hi]).reshape(lead + self.grid)
        return out

    def steps(self, state, n):
        seen = []
        with torch.no_grad():
            for k in range(n):
                state, s = self.step(state, k)
                seen.append(s)
        return state, torch.stack(seen)


def _zero(sim):
    nd = len(sim.shape)
    z = torch.zeros(tuple(sim.shape[::-1]), dtype=torch.float64, device=DEV)
    return tuple(z for _ in range(1 + nd + 2 * nd * sim.n_relax))


def _exact_gradient(sim, state, weights, n):
    """Gradient of the misfit (weights None: observed traces in obs) or of
    sum(weights * trace) over n steps with respect to c."""
    c = torch.as_tensor(sim.c, dtype=torch.float64, device=DEV).requires_grad_(True)
    e = _Exact(sim, c)

    def one(k, *s):
        new, seen = e.step(s, k)
        return (seen,) + new

    J = 0.0
    for k in range(n):
        got = checkpoint(one, k, *state, use_reentrant=False)
        J = J + weights(k, got[0])
        state = got[1:]
    J.backward()
    return J.detach(), c.grad


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        sims, n = _batch_simulations(case, seed), case["n"]
        traces, fields = [], []
        for k, sim in enumerate(sims):
            e = _Exact(sim)
            state, seen = e.steps(e.split(_state(sim, seed + k)), n)
            traces.append(seen)
            fields.append(e.packed(state, fw2.FIELD_P))
        return traces[:16] + fields
    if kind in ("gradient", "reverse"):
        sim, obs = _observed(case, seed)
        w = torch.as_tensor(obs, dtype=torch.float64, device=DEV)
        if kind == "gradient":
            J, g = _exact_gradient(sim, _zero(sim), lambda k, s: 0.5 * ((s - w[k]) ** 2).sum(), case["n"])
            return {"misfit": J, "gradient": g}
        state = tuple(x.clone() for x in _Exact(sim).split(_state(sim, seed)))
        return _exact_gradient(sim, state, lambda k, s: (s * w[k]).sum(), case["n"])[1]
    sim = _case_simulation(case, seed)
    e = _Exact(sim)
    start = e.split(_state(sim, seed) if kind != "slabs" else _slab_state(case, sim, seed)[1])
    n = {"poll": 1, "checkpoint": 1}.get(kind) or case["n"]
    state, seen = e.steps(start, n)
    if kind == "event":
        return {"trace": seen, **e.packed(state, FIELDS[case["read"]])}
    if kind == "slabs":
        bounds, f = _slab_state(case, sim, seed)[0], e.packed(state, FIELDS["pv"])
        return [{q: f[q].narrow(-3, a, b - a).contiguous() for q in f} for a, b in zip(bounds, bounds[1:])]
    return e.packed(state, fw2.FIELD_P if kind == "poll" else fw2.FIELD_ALL)
