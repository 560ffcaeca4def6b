"""The work whose speed is followed: what a user of this framework has it do.

Every case goes through the package's public entry points (`Problem`,
`DeviceState`, `fit.Loop`, `autograd.prism_loss`, `rprop_step_ptr`) on seeded
synthetic measurements of the shapes that the package's workloads, tests and
benchmark use.  `listed()` are the cases followed by name, `draw(rng)` gives
further ones of the same ranges, `prepare` builds what a program holds before
the call, `run` is one call, `work` what the call cannot do without, and
`exact` the outputs in float64 from plain torch.

The entry points, by the case's "op":
  adam      DeviceState.iteration(): one Adam iteration of a fit, in place
  graph     the same iteration captured as a HIP graph (fit.Loop), one replay
  autograd  prism_loss(): the loss and its gradient through torch.autograd
  synth     DeviceState.synthesize(): the forward model alone
  stitch    DeviceState.stitch_maps(): per-slab maps blended into a volume
  rprop     rprop_step_ptr(): the paper's optimiser on a gradient in hand

The fit's state is that of a running fit: parameters near the measured
tissue, moments of earlier steps, step counter above zero.  The loss terms are
sums of FP32 terms, kept in FP64 between iterations by the library; the
outputs give them in FP32.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

LR, BETA1, BETA2, EPS = 1e-2, 0.9, 0.999, 1e-8
RPROP = (0.5, 1.2, 1e-6, 50.0)
STEPS_DONE = 20                     # optimiser steps before the measured one
# model constants (the library's defaults)
D_CSF, D_GM, D_RES, D_PAR, D_PERP = 3.0, 0.9, 0.2, 1.7, 0.4
LAM = dict(spatial=0.01, rep=0.01, sparse=0.02, orphan=0.01, continuity=0.005, ordering=0.01, tv=0.01, cal=0.01)
HUBER, TAU, S0_ORPHAN = 0.05, 0.15, 0.1
TERMS = ("data", "spatial", "rep", "sparse", "orphan", "continuity", "ordering", "cal", "tv")
STANDARD = "spatial,rep,sparse,cal"
EVERY = "spatial,rep,sparse,cal,orphan,continuity,ordering,tv"
N_BIAS = {"none": 0, "poly2": 10, "trilinear8": 512}


def _case(name, op, nx, ny, nz, **kw):
    c = dict(op=op, nx=nx, ny=ny, nz=nz, brain=False, n_b0=1, shells=1, first_shell=1, per_shell=32,
             interleaved=False, K=3, nll=False, bias="none", learn_d=False, neighbourhood=6, priors=STANDARD,
             snr=30.0, slabs=False, groups=1, persistent=False)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one 8^3 patch of crossing fibres: the smallest fit, replayed as a graph for a
        # hundred iterations; all latency
        _case("patch8_graph", "graph", 8, 8, 8, priors="rep"),
        # one 16^3 multi-shell patch with calibration under the Rician likelihood, stepped
        # eagerly (a program that looks at the fit between iterations)
        _case("patch16_nll_adam", "adam", 16, 16, 16, n_b0=18, shells=3, per_shell=90, nll=True, bias="poly2"),
        # the crossing-fibre benchmark (16 angles and single fibres, 200 voxels each),
        # differentiated through autograd for an outside optimiser
        _case("crossings_nll_autograd", "autograd", 17, 200, 1, shells=3, per_shell=64, K=2, nll=True,
              neighbourhood=0, priors="rep,sparse,cal"),
        # the 40^3 bundle phantom: four fibres, learned diffusivities and noise level
        _case("phantom_learned_d_adam", "adam", 40, 40, 40, n_b0=6, shells=2, per_shell=45, K=4, nll=True,
              bias="poly2", learn_d=True, snr=20.0),
        # twenty axial slices of a single-shell scan, measurements in scanner order (the b = 0
        # images spread through the series)
        _case("hardi_slices_graph", "graph", 81, 106, 20, brain=True, n_b0=10, shells=1, first_shell=2,
              per_shell=150, interleaved=True, bias="poly2"),
        # every term of the objective at once: the 8^3 bias grid with its total variation, the
        # 26-neighbourhood, the stabilisation priors; odd edges
        _case("all_priors_nll_adam", "adam", 63, 59, 37, brain=True, shells=3, per_shell=64, nll=True,
              bias="trilinear8", neighbourhood=26, priors=EVERY),
        # the whole-brain-shaped volume as one problem
        _case("brain_adam", "adam", 145, 174, 145, brain=True, n_b0=18, shells=3, per_shell=90, bias="poly2"),
        # the same volume as 30-slice slabs with 5-slice overlaps, fitted together; the shells
        # interleaved as scanners acquire them
        _case("brain_slabs_adam", "adam", 145, 174, 145, brain=True, n_b0=6, shells=2, per_shell=45, K=2,
              interleaved=True, bias="poly2", slabs=True),
        # the slabs' maps blended into whole-volume maps
        _case("brain_stitch", "stitch", 145, 174, 145, brain=True, slabs=True, bias="poly2"),
        # the fitted model's signal for the whole volume (residual maps, simulation)
        _case("brain_synth", "synth", 145, 174, 145, brain=True, n_b0=18, shells=3, per_shell=90, bias="poly2"),
        # Rprop's update of the volume's parameters
        _case("brain_rprop", "rprop", 145, 174, 145, brain=True, bias="poly2"),
        # many small independent patches, every fibre count, likelihood and protocol mixed, in
        # the plan that the autotuner picks for such batches
        _case("patches_mixed_adam", "adam", 4, 24, 0, groups=512, persistent=True),
    ]


def draw(rng):
    """One more case of the ranges above."""
    def span(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["graph", "adam", "adam", "adam", "autograd", "synth", "stitch", "rprop", "batch"])
    n_b0, shells = rng.randint(1, 18), rng.randint(1, 3)
    kw = dict(n_b0=n_b0, shells=shells, first_shell=2 if shells == 1 and rng.random() < 0.5 else 1,
              per_shell=span(24, 90), interleaved=rng.random() < 0.5, K=rng.randint(1, 5), nll=rng.random() < 0.4,
              bias=rng.choice(["none", "poly2", "poly2", "trilinear8"]), learn_d=rng.random() < 0.2,
              neighbourhood=rng.choice([0, 6, 6, 6, 26]), snr=float(rng.choice([10, 20, 30, 50])),
              priors=rng.choice(["rep", "rep,sparse,cal", STANDARD, STANDARD, STANDARD, EVERY]))
    if op == "batch":
        return _case(None, "adam", 4, rng.randint(8, 24), 0, groups=span(24, 512), persistent=rng.random() < 0.5)
    if op in ("stitch", "rprop"):
        e = span(40, 150)
        return _case(None, op, e, max(8, e + rng.randint(-9, 24)), max(24, e - rng.randint(0, 9)), brain=True,
                     slabs=op == "stitch", K=kw["K"], learn_d=kw["learn_d"], bias="poly2")
    # box volumes from one 8^3 patch to the volume; no more pairs (times their cost) than the
    # volume's fit
    e = span(7, 110)
    nx, ny, nz = max(3, e + rng.randint(-3, 3)), max(3, e + rng.randint(-3, 9)), max(2, e - rng.randint(0, 5))
    n = n_b0 + shells * kw["per_shell"]
    cost = nx * ny * nz * n * (kw["K"] + 2.0) * (3.0 if kw["nll"] else 1.0) * (1.5 if kw["learn_d"] else 1.0)
    if cost > 6e8:
        kw.update(nll=False, learn_d=False, K=min(kw["K"], 3))
    return _case(None, op, nx, ny, nz, brain=rng.random() < 0.5,
                 slabs=op == "adam" and nz >= 31 and rng.random() < 0.3, **kw)


# ----------------------------------------------------------------------------
# the groups of a case, their acquisitions and masks (host)
# ----------------------------------------------------------------------------

class _Group:
    """One independent problem of a case: box, mask, acquisition and options."""

    def __init__(self, c, shape, mask, bval, bvec, **over):
        self.shape, self.mask, self.bval, self.bvec = shape, mask, bval, bvec
        for k in ("K", "nll", "bias", "learn_d", "neighbourhood", "snr"):
            setattr(self, k, over.get(k, c[k]))
        self.priors = tuple(c["priors"].split(","))
        self.V, self.N = int(mask.sum()), int(bval.shape[0])
        self.C = self.K + 3
        self.P = 5 + 4 * self.K + (2 if self.learn_d else 0)
        self.n_bias = N_BIAS[self.bias]
        self.n_cal = self.n_bias + 2 * self.N + 1


def _acquisition(n_b0, shells, first_shell, per_shell, interleaved, rng):
    b = np.concatenate([np.zeros(n_b0)] + [np.full(per_shell, float(first_shell + i)) for i in range(shells)])
    g = rng.standard_normal((b.size, 3))
    g /= np.linalg.norm(g, axis=1, keepdims=True)
    g[b == 0.0] = (1.0, 0.0, 0.0)
    if interleaved:
        order = np.concatenate([[0], 1 + rng.permutation(b.size - 1)])    # a b = 0 image comes first
        b, g = b[order], g[order]
    return b, g


def _mask(c, rng):
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    if not c["brain"]:
        return np.ones((nx, ny, nz), dtype=bool)
    # an ellipsoid of about a fifth of the box, as the brain-shaped volume's (nearly the box
    # across thin ones)
    ax = [(np.arange(n) - (n - 1) / 2.0 - rng.uniform(-0.5, 0.5)) / (0.363 * n + 0.5) for n in (nx, ny, nz)]
    if nz <= 24:
        ax[2] = 0.5 * ax[2]
    return ax[0][:, None, None] ** 2 + ax[1][None, :, None] ** 2 + ax[2][None, None, :] ** 2 <= 1.0


def _groups(case, seed):
    rng = np.random.default_rng([seed, 11])
    if case["groups"] > 1:
        acqs = [_acquisition(n0, sh, 1, per, False, rng) for n0, sh, per in ((1, 1, 32), (6, 2, 45), (18, 3, 90))]
        # sizes, protocols and options are the case's, the same for every seed
        plan = np.random.default_rng([case["groups"], case["ny"], 13])
        out = []
        for _ in range(case["groups"]):
            e = int(round(math.exp(plan.uniform(math.log(case["nx"]), math.log(case["ny"])))))
            bval, bvec = acqs[int(plan.integers(0, 3))]
            out.append(_Group(case, (e, e, e), np.ones((e, e, e), dtype=bool), bval, bvec, K=int(plan.integers(1, 6)),
                              nll=bool(plan.random() < 0.5), snr=float(plan.uniform(10.0, 50.0))))
        return out, None
    bval, bvec = _acquisition(case["n_b0"], case["shells"], case["first_shell"], case["per_shell"],
                              case["interleaved"], rng)
    mask = _mask(case, np.random.default_rng(case["nx"]))
    if not case["slabs"]:
        return [_Group(case, mask.shape, mask, bval, bvec)], None
    starts, nz = [0], mask.shape[2]
    while starts[-1] + 30 < nz:
        starts.append(starts[-1] + 25)
    return [_Group(case, (mask.shape[0], mask.shape[1], min(30, nz - z)), mask[:, :, z:z + 30].copy(), bval, bvec)
            for z in starts], starts


# ----------------------------------------------------------------------------
# seeded measurements and fit state (on the GPU)
# ----------------------------------------------------------------------------

def _unit(x, dim):
    return x / x.norm(dim=dim, keepdim=True)


def _tissue(V, n_fib, gen, dev):
    """Ground truth of V voxels: Dirichlet fractions (csf, gm, res, fibres), fibre
    directions and tensor diffusivities."""
    w = torch.empty(3 + n_fib, V, device=dev).exponential_(generator=gen)
    u = _unit(torch.randn(n_fib, 3, V, device=dev, generator=gen), 1)
    dpar = 1.5 + 0.7 * torch.rand(n_fib, V, device=dev, generator=gen)
    dperp = 0.3 + 0.4 * torch.rand(n_fib, V, device=dev, generator=gen)
    return w / w.sum(0, keepdim=True), u, dpar, dperp


def _measure(g, tissue, gen, dev, out):
    """Rician measurements of the tissue into out [N, V]."""
    frac, u, dpar, dperp = tissue
    b = torch.tensor(g.bval, dtype=torch.float32, device=dev)[:, None]
    G = torch.tensor(g.bvec, dtype=torch.float32, device=dev)
    step = max(1, (1 << 23) // g.N)
    for lo in range(0, g.V, step):
        s = slice(lo, min(g.V, lo + step))
        S = frac[0, s] * torch.exp(-3.0 * b) + frac[1, s] * torch.exp(-0.8 * b) + frac[2, s] * torch.exp(-0.1 * b)
        for k in range(u.shape[0]):
            q = (G @ u[k][:, s]).square_()
            S += frac[3 + k, s] * torch.exp(-b * (dperp[k, s] + (dpar[k, s] - dperp[k, s]) * q))
        n1 = torch.randn(S.shape, device=dev, generator=gen) / g.snr
        n2 = torch.randn(S.shape, device=dev, generator=gen) / g.snr
        out[:, s] = torch.hypot(S + n1, n2)


def _theta(g, tissue, gen, dev):
    """Raw parameter rows [P, V] near the tissue, as some way into a fit."""
    def normal(scale, *shape):
        return scale * torch.randn(*shape, device=dev, generator=gen)

    frac, u, _, _ = tissue
    th = torch.empty(g.P, g.V, device=dev)
    th[0] = math.log(math.e - 1.0) + normal(0.1, g.V)
    order = [0, 1] + [3 + min(k, u.shape[0] - 1) for k in range(g.K)] + [2]
    for row, c in enumerate(order):
        th[1 + row] = torch.log(frac[c] + 0.02) + normal(0.2, g.V)
    for k in range(g.K):
        d = u[k] if k < u.shape[0] else _unit(normal(1.0, 3, g.V), 0)
        th[1 + g.C + 3 * k:4 + g.C + 3 * k] = (_unit(d + normal(0.2, 3, g.V), 0)
                                               * (1.0 + 0.2 * torch.rand(g.V, device=dev, generator=gen)))
    th[1 + g.C + 3 * g.K] = normal(0.5, g.V)
    if g.learn_d:
        th[g.P - 2] = math.log(math.expm1(1.7)) + normal(0.2, g.V)
        th[g.P - 1] = math.log(math.expm1(0.4)) + normal(0.2, g.V)
    return th


def _cal(g, gen, dev):
    cal = torch.empty(g.n_cal, device=dev)
    cal[:g.n_bias].normal_(0.0, 0.04, generator=gen)
    cal[g.n_bias:g.n_bias + g.N].normal_(0.0, 0.03, generator=gen)
    cal[g.n_bias + g.N:g.n_bias + 2 * g.N].normal_(0.0, 0.01, generator=gen)
    cal[-1] = math.log(1.5 / g.snr) if g.nll else 0.0
    return cal


def _gradient_scale(g):
    """Size of a voxel's and of a calibration parameter's gradient (noise-level residuals)."""
    r = (1.0 / g.snr if not g.nll else g.snr) * 0.3
    m = 2.0 / g.V if not g.nll else 1.0
    return m * r * math.sqrt(g.N), m * r * math.sqrt(g.V)


def _inputs(case, seed, dev, need_y=True, need_moments=True):
    """Groups, slab starts and the flat buffers [theta_micro | theta_cal], y, moments."""
    groups, starts = _groups(case, seed)
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed * 7919 + 17)
    n_micro, n_cal = sum(g.P * g.V for g in groups), sum(g.n_cal for g in groups)
    params = torch.empty(n_micro + n_cal, device=dev)
    y = torch.empty(sum(g.N * g.V for g in groups), device=dev) if need_y else None
    m = torch.empty_like(params) if need_moments else None
    v = torch.empty_like(params) if need_moments else None
    a, b, c = 0, n_micro, 0
    previous = None
    for i, g in enumerate(groups):
        tissue = _tissue(g.V, 3, gen, dev)
        if previous is not None:
            # a slab sees the tissue of the slab below in the five slices they share
            below, z = previous
            for t, old in zip(tissue, z):
                t[..., _slices(g, 0, 5)] = old[..., _slices(below, 25, 30)]
        if starts is not None:
            previous = (g, tissue)
        params[a:a + g.P * g.V].view(g.P, g.V)[:] = _theta(g, tissue, gen, dev)
        params[b:b + g.n_cal] = _cal(g, gen, dev)
        if need_y:
            _measure(g, tissue, gen, dev, y[c:c + g.N * g.V].view(g.N, g.V))
        if need_moments:
            for lo, n, s in ((a, g.P * g.V, _gradient_scale(g)[0]), (b, g.n_cal, _gradient_scale(g)[1])):
                m[lo:lo + n].normal_(0.0, 0.7 * s, generator=gen)
                v[lo:lo + n] = (s * (0.5 + torch.rand(n, device=dev, generator=gen))).square_()
        a, b, c = a + g.P * g.V, b + g.n_cal, c + g.N * g.V
    return groups, starts, params, y, m, v


def _slices(g, lo, hi):
    """Indices of the group's voxels in its slices lo..hi-1, in raster order."""
    z = np.nonzero(g.mask)[2]
    return torch.from_numpy(np.nonzero((z >= lo) & (z < hi))[0])


# ----------------------------------------------------------------------------
# the call
# ----------------------------------------------------------------------------

def prepare(case, seed):
    from paper_2604_00250_amd import inputs as I
    from paper_2604_00250_amd.fit import Loop, restore, snapshot
    from paper_2604_00250_amd.problem import DeviceState, Problem

    dev = torch.device("cuda:0")
    op = case["op"]
    if op == "rprop":
        n, g, p, prev, step = _rprop_inputs(case, seed, dev)
        return dict(op=op, n=n, g=g, p=p, prev=prev, step=step)
    stepped = op in ("adam", "graph")
    groups, starts, params, y, m, v = _inputs(case, seed, dev, op in ("adam", "graph", "autograd"), stepped)
    acqs = {}
    described = []
    for g in groups:
        if id(g.bval) not in acqs:
            acqs[id(g.bval)] = I.Acquisition(bval=g.bval, bvec=g.bvec)
        described.append(I.Group(shape=g.shape, mask=g.mask, acq=acqs[id(g.bval)], K=g.K,
                                 mode="nll" if g.nll else "mse", bias=g.bias, learn_diffusivity=g.learn_d,
                                 neighbourhood=g.neighbourhood, priors=g.priors))
    launch = dict(vox_per_lane=1, n_split=0, item_vox=0, persistent=1) if case["persistent"] else None
    prob = Problem(described, launch=launch)
    st = DeviceState(prob)
    st.params.copy_(params)
    if y is not None:
        st.y.copy_(y)
    state = dict(op=op, st=st)
    if stepped:
        st.m.copy_(m)
        st.v.copy_(v)
        st.step[0] = STEPS_DONE
        n = st.n_micro
        state["out"] = dict(theta_micro=st.params[:n], theta_cal=st.params[n:], m_micro=st.m[:n], m_cal=st.m[n:],
                            v_micro=st.v[:n], v_cal=st.v[n:])
    if op == "graph":
        loop = Loop(st, lr=LR, history=100)
        snap = snapshot(st)
        loop.capture()
        restore(st, snap)
        state["loop"] = loop
    elif op == "autograd":
        state["params"] = st.params.clone().requires_grad_(True)
    elif op == "stitch":
        prob.stitch_plan((case["nx"], case["ny"], case["nz"]), starts)
    return state


def run(state):
    op = state["op"]
    if op == "rprop":
        from paper_2604_00250_amd import rprop_step_ptr
        p, g, prev, step = state["p"], state["g"], state["prev"], state["step"]
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        rprop_step_ptr(p.data_ptr(), g.data_ptr(), prev.data_ptr(), step.data_ptr(), state["n"], *RPROP, stream)
        return dict(p=p, prev=prev, step=step)
    st = state["st"]
    if op == "adam":
        st.iteration(lr=LR)
        return dict(state["out"], loss=st.loss.float())
    if op == "graph":
        state["loop"].replay(1)
        return dict(state["out"], loss=st.loss.float())
    if op == "autograd":
        from paper_2604_00250_amd.autograd import prism_loss
        loss = prism_loss(state["params"], st)
        (grad,) = torch.autograd.grad(loss, state["params"])
        return dict(loss=loss.detach().float(), g_micro=grad[:st.n_micro], g_cal=grad[st.n_micro:])
    if op == "synth":
        return st.synthesize()
    return st.stitch_maps()


def work(case):
    """Bytes: each input read once, each output written once.  Operations: the pass's
    algebra per (voxel, measurement) with a fibre's attenuation as two exponentials
    (forward 7K + 3 multiply-adds, adjoint 8K + 7, data term 3; 30 more for the Rician
    terms, 6K for learned diffusivities), two operations each."""
    groups, starts = _groups(case, 0)
    b = f = 0.0
    if case["op"] == "rprop":
        n = sum(g.P * g.V + g.n_cal for g in groups)
        return {"bytes": 4.0 * 7 * n, "flops": 5.0 * n}
    if case["op"] == "stitch":
        out = int(_mask(case, np.random.default_rng(case["nx"])).sum())
        g0 = groups[0]
        inside = sum(g.V for g in groups)
        return {"bytes": 4.0 * g0.P * (inside + out) + 24.0 * out, "flops": 30.0 * g0.P * out}
    for g in groups:
        pairs = g.V * g.N
        fwd = 7 * g.K + 3
        if case["op"] == "synth":
            b += 4.0 * g.N * g.V + 4.0 * g.P * g.V
            f += 2.0 * pairs * (fwd + 1) + 2.0 * g.K * pairs
            continue
        adj = 8 * g.K + 7 + (6 * g.K if g.learn_d else 0)
        f += pairs * (2.0 * (fwd + adj + (33 if g.nll else 3)) + 2.0 * g.K)
        rows = 6 if case["op"] in ("adam", "graph") else 2       # theta, m, v in and out; theta in, gradient out
        b += 4.0 * g.N * g.V + 4.0 * rows * (g.P * g.V + g.n_cal)
    return {"bytes": b, "flops": f}


# ----------------------------------------------------------------------------
# the outputs in float64, from plain torch
# ----------------------------------------------------------------------------

def _rprop_inputs(case, seed, dev):
    groups, _ = _groups(case, seed)
    n = sum(g.P * g.V + g.n_cal for g in groups)
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed * 7919 + 17)
    s = _gradient_scale(groups[0])[0]
    p = torch.randn(n, device=dev, generator=gen)
    prev = s * torch.randn(n, device=dev, generator=gen)
    g = 0.6 * prev + 0.8 * s * torch.randn(n, device=dev, generator=gen)
    prev *= torch.rand(n, device=dev, generator=gen) > 0.1       # coordinates that flipped in the last step
    step = LR * torch.exp(torch.randn(n, device=dev, generator=gen))
    return n, g, p, prev, step


def _box_index(g, dev):
    """Voxel of each box position, padded by one on every side (V: none), and the
    voxels' positions in the padded box."""
    coords = np.argwhere(g.mask)
    pad = [n + 2 for n in g.shape]
    at = torch.from_numpy(np.ravel_multi_index((coords + 1).T, pad)).to(dev)
    box = torch.full((pad[0] * pad[1] * pad[2],), g.V, dtype=torch.int64, device=dev)
    box[at] = torch.arange(g.V, device=dev)
    return box, at, pad, torch.from_numpy(coords).to(dev).double()


def _offsets(neighbourhood):
    near = [(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1) if (a, b, c) != (0, 0, 0)]
    return near if neighbourhood == 26 else [o for o in near if sum(map(abs, o)) == 1]


def _log_bias(g, coords, w):
    """log B of the voxels at box coordinates `coords` from the basis coefficients."""
    if g.bias == "poly2":
        x, y, z = (((2.0 * coords[:, a] - (n - 1)) / (n - 1)) if n > 1 else 0.0 * coords[:, a]
                   for a, n in enumerate(g.shape))
        return (w[0] + w[1] * x + w[2] * y + w[3] * z + w[4] * x * x + w[5] * y * y + w[6] * z * z + w[7] * x * y
                + w[8] * x * z + w[9] * y * z)
    cell, frac = [], []
    for a, n in enumerate(g.shape):
        p = coords[:, a] * (7.0 / (n - 1)) if n > 1 else 0.0 * coords[:, a]
        i = p.floor().clamp(max=6).long()
        cell.append(i)
        frac.append(p - i)
    out = 0.0
    for cx in (0, 1):
        for cy in (0, 1):
            for cz in (0, 1):
                weight = 1.0
                for a, o in enumerate((cx, cy, cz)):
                    weight = weight * (frac[a] if o else 1.0 - frac[a])
                out = out + weight * w[((cell[0] + cx) * 8 + cell[1] + cy) * 8 + cell[2] + cz]
    return out


def _constrain(g, th):
    S0 = torch.nn.functional.softplus(th[0], threshold=100.0)
    f = torch.softmax(th[1:1 + g.C], 0)
    v = th[1 + g.C:1 + g.C + 3 * g.K].reshape(g.K, 3, -1)
    d = v / v.square().sum(1, keepdim=True).sqrt()
    fin = torch.sigmoid(th[1 + g.C + 3 * g.K])
    if g.learn_d:
        D = [torch.nn.functional.softplus(th[g.P - 2 + i], threshold=100.0) for i in (0, 1)]
    else:
        D = [D_PAR, D_PERP]
    return S0, f, d, fin, D


def _signal(g, th, log_b, alpha, beta, bval, bvec):
    S0, f, d, fin, (dpar, dperp) = _constrain(g, th)
    S = f[0] * torch.exp(-D_CSF * bval) + f[1] * torch.exp(-D_GM * bval) + f[g.C - 1] * torch.exp(-D_RES * bval)
    for k in range(g.K):
        c2 = (bvec @ d[k]).square()
        stick = torch.exp(-bval * dpar * c2)
        S = S + f[2 + k] * stick * (fin + (1.0 - fin) * torch.exp(-bval * dperp * (1.0 - c2)))
    return torch.exp(alpha)[:, None] * (torch.exp(log_b) * S0) * S + beta[:, None]


def _split_cal(g, cal):
    return cal[:g.n_bias], cal[g.n_bias:g.n_bias + g.N], cal[g.n_bias + g.N:g.n_bias + 2 * g.N], cal[-1]


def _data_loss(g, yhat, y, sigma_log):
    if not g.nll:
        return (yhat - y).square().sum() / g.V
    s2 = torch.exp(2.0 * sigma_log)
    z = (y * yhat).abs() / s2
    log_i0 = z + torch.log(torch.special.i0e(z))
    return (2.0 * sigma_log + (y * y + yhat * yhat) / (2.0 * s2) - log_i0).sum()


def _prior_losses(g, th, cal, box, at, pad, coords):
    """The terms that couple voxels or act on a voxel's parameters alone."""
    S0, f, d, _, _ = _constrain(g, th)
    w, alpha, beta, _ = _split_cal(g, cal)
    fw, on, V = f[2:2 + g.K], set(g.priors), g.V
    out = {}

    def neighbours(offset):
        return box[at + (offset[0] * pad[1] + offset[1]) * pad[2] + offset[2]]

    def padded(x):
        return torch.cat([x, torch.zeros_like(x[..., :1])], -1)

    if g.neighbourhood:
        count = sum((neighbours(o) < V).double() for o in _offsets(g.neighbourhood))
        inv = torch.where(count > 0, 1.0 / count.clamp(min=1.0), 0.0 * count)
    if "spatial" in on and g.neighbourhood:
        fp = padded(f)
        mean = sum(fp[:, neighbours(o)] for o in _offsets(g.neighbourhood)) * inv
        a = torch.where(count > 0, f - mean, 0.0 * f).abs()
        out["spatial"] = torch.where(a <= HUBER, 0.5 * a * a, HUBER * (a - 0.5 * HUBER)).sum()
    if "rep" in on:
        out["rep"] = sum(((fw[i] * fw[j] * (d[i] * d[j]).sum(0).abs()).sum() for i in range(g.K)
                          for j in range(i + 1, g.K)), 0.0 * S0.sum())
    if "sparse" in on:
        out["sparse"] = (fw * (fw.detach() < TAU)).sum()
    if "orphan" in on:
        out["orphan"] = ((1.0 - S0 / S0_ORPHAN).clamp(min=0.0) * fw.sum(0)).sum()
    if "continuity" in on and g.neighbourhood:
        dp, total = padded(d), 0.0
        for o in _offsets(g.neighbourhood):
            u = neighbours(o)
            total = total + (inv * (u < V) * (1.0 - (d * dp[:, :, u]).sum(1).square()).sum(0)).sum()
        out["continuity"] = total
    if "ordering" in on:
        out["ordering"] = (fw[1:] - fw[:-1]).clamp(min=0.0).sum()
    if "tv" in on and g.bias != "none":
        B = torch.exp(_log_bias(g, coords, w))
        Bp = padded(B)
        out["tv"] = sum((((neighbours(o) < V) * (Bp[neighbours(o)] - B)).abs()).sum()
                        for o in ((1, 0, 0), (0, 1, 0), (0, 0, 1)))
    out = {k: LAM[k] / V * x for k, x in out.items()}
    if "cal" in on:
        out["cal"] = LAM["cal"] * (alpha.square().sum() + beta.square().sum() + w.square().sum())
    return out


def _loss_and_gradient(g, th, cal, y, dev):
    """Loss terms [10] and the gradients of the total, all float64."""
    th, cal = th.double().requires_grad_(True), cal.double().requires_grad_(True)
    box, at, pad, coords = _box_index(g, dev)
    bval = torch.tensor(g.bval, device=dev).float().double()[:, None]
    bvec = torch.tensor(g.bvec, device=dev).float().double()
    losses = dict.fromkeys(TERMS, 0.0)
    step = max(1, (1 << 21) // g.N)
    g_th, g_cal = torch.zeros_like(th), torch.zeros_like(cal)
    for lo in range(0, g.V, step):
        s = slice(lo, min(g.V, lo + step))
        part = th.detach()[:, s].clone().requires_grad_(True)
        w, alpha, beta, sigma_log = _split_cal(g, cal)
        log_b = _log_bias(g, coords[s], w) if g.n_bias else torch.zeros_like(part[0])
        yhat = _signal(g, part, log_b, alpha, beta, bval, bvec)
        loss = _data_loss(g, yhat, y[:, s].double(), sigma_log)
        gt, gc = torch.autograd.grad(loss, (part, cal))
        g_th[:, s] = gt
        g_cal += gc
        losses["data"] += float(loss.detach())
    terms = _prior_losses(g, th, cal, box, at, pad, coords)
    total = sum(terms.values(), 0.0 * (th[0].sum() + cal.sum()))
    gt, gc = torch.autograd.grad(total, (th, cal), allow_unused=True)
    losses.update({k: float(x.detach()) for k, x in terms.items()})
    row = [losses[t] for t in TERMS]
    return row + [sum(row)], g_th + gt, g_cal + gc


def _stitched(case, groups, starts, params, dev):
    maps, w, cells = [], [], []
    a = 0
    nz = case["nz"]
    for i, g in enumerate(groups):
        th = params[a:a + g.P * g.V].view(g.P, g.V).double()
        a += g.P * g.V
        S0, f, d, fin, D = _constrain(g, th)
        maps.append(torch.cat([S0[None], f, d.reshape(3 * g.K, -1), fin[None]] + ([x[None] for x in D] if g.learn_d else [])))
        c = torch.from_numpy(np.argwhere(g.mask)).to(dev)
        t = g.shape[2]
        low = max(0, starts[i - 1] + groups[i - 1].shape[2] - starts[i]) if i else 0
        high = max(0, starts[i] + t - starts[i + 1]) if i + 1 < len(groups) else 0
        z = c[:, 2].double()
        weight = torch.ones_like(z)
        if low:
            weight = torch.minimum(weight, (z + 1.0) / (low + 1.0))
        if high:
            weight = torch.minimum(weight, (t - z) / (high + 1.0))
        w.append(weight)
        cells.append((c[:, 0] * case["ny"] + c[:, 1]) * nz + starts[i] + c[:, 2])
    g0, C = groups[0], groups[0].C
    out = torch.zeros(g0.P, case["nx"] * case["ny"] * nz, dtype=torch.float64, device=dev)
    weight = torch.zeros(out.shape[1], dtype=torch.float64, device=dev)
    for x, wx, at in zip(maps, w, cells):
        both = weight[at] > 0
        fresh = at[~both]
        out[:, fresh], weight[fresh] = x[:, ~both], wx[~both]
        if not bool(both.any()):
            continue
        p = at[both]
        wl, wu = weight[p], wx[both]
        wl, wu = wl / (wl + wu), wu / (wl + wu)
        lower, upper = out[:, p], x[:, both]
        first = wl >= wu
        r, q = torch.where(first, lower, upper), torch.where(first, upper, lower)
        wr, wo = torch.where(first, wl, wu), torch.where(first, wu, wl)
        res = wr * r + wo * q
        dr = r[1 + C:1 + C + 3 * g0.K].reshape(g0.K, 3, -1)
        dq = q[1 + C:1 + C + 3 * g0.K].reshape(g0.K, 3, -1)
        dots = torch.stack([torch.stack([(dr[k] * dq[j]).sum(0) for j in range(g0.K)]) for k in range(g0.K)])
        free = torch.ones_like(dots[0], dtype=torch.bool)
        pick = torch.arange(p.numel(), device=dev)
        for k in range(g0.K):
            j = torch.where(free, dots[k].abs(), -torch.ones_like(dots[k])).argmax(0)
            free[j, pick] = False
            sign = torch.where(dots[k][j, pick] < 0, -1.0, 1.0)
            res[3 + k] = wr * r[3 + k] + wo * q[3 + j, pick]
            e = wr * dr[k] + wo * sign * dq[j, :, pick].T
            res[1 + C + 3 * k:4 + C + 3 * k] = e / e.norm(dim=0)
        out[:, p] = res
    return out[:, weight > 0]


def exact(case, seed):
    dev = torch.device("cuda:0" if torch.cuda.is_available() else "cpu")
    op = case["op"]
    if op == "rprop":
        _, g, p, prev, step = (x.double() if torch.is_tensor(x) else x for x in _rprop_inputs(case, seed, dev))
        s = g * prev
        step = (step * torch.where(s > 0, RPROP[1], torch.where(s < 0, RPROP[0], torch.ones_like(s)))).clamp(*RPROP[2:])
        g = torch.where(s < 0, 0.0 * g, g)
        return dict(p=p - torch.sign(g) * step, prev=g, step=step)
    stepped = op in ("adam", "graph")
    groups, starts, params, y, m, v = _inputs(case, seed, dev, op in ("adam", "graph", "autograd"), stepped)
    if op == "stitch":
        return _stitched(case, groups, starts, params, dev)
    n_micro = sum(g.P * g.V for g in groups)
    if op == "synth":
        g = groups[0]
        out = torch.empty(g.N * g.V, dtype=torch.float64, device=dev)
        th, cal = params[:n_micro].view(g.P, g.V).double(), params[n_micro:].double()
        coords = torch.from_numpy(np.argwhere(g.mask)).to(dev).double()
        w, alpha, beta, _ = _split_cal(g, cal)
        bval = torch.tensor(g.bval, device=dev).float().double()[:, None]
        bvec = torch.tensor(g.bvec, device=dev).float().double()
        step = max(1, (1 << 23) // g.N)
        for lo in range(0, g.V, step):
            s = slice(lo, min(g.V, lo + step))
            log_b = _log_bias(g, coords[s], w) if g.n_bias else torch.zeros_like(th[0, s])
            out.view(g.N, g.V)[:, s] = _signal(g, th[:, s], log_b, alpha, beta, bval, bvec)
        return out
    grad = torch.empty_like(params, dtype=torch.float64)
    rows, a, b, c = [], 0, n_micro, 0
    for g in groups:
        row, gt, gc = _loss_and_gradient(g, params[a:a + g.P * g.V].view(g.P, g.V), params[b:b + g.n_cal],
                                         y[c:c + g.N * g.V].view(g.N, g.V), dev)
        rows.append(row)
        grad[a:a + g.P * g.V] = gt.reshape(-1)
        grad[b:b + g.n_cal] = gc
        a, b, c = a + g.P * g.V, b + g.n_cal, c + g.N * g.V
    loss = torch.tensor(rows, dtype=torch.float64, device=dev)
    if op == "autograd":
        return dict(loss=loss[:, -1].sum(), g_micro=grad[:n_micro], g_cal=grad[n_micro:])
    t = STEPS_DONE + 1
    m = BETA1 * m.double() + (1.0 - BETA1) * grad
    v = BETA2 * v.double() + (1.0 - BETA2) * grad * grad
    p = params.double() - LR / (1.0 - BETA1 ** t) * m / (v.sqrt() / math.sqrt(1.0 - BETA2 ** t) + EPS)
    return dict(theta_micro=p[:n_micro], theta_cal=p[n_micro:], m_micro=m[:n_micro], m_cal=m[n_micro:],
                v_micro=v[:n_micro], v_cal=v[n_micro:], loss=loss)
