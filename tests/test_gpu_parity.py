"""GPU parity of the HIP path (through the C ABI) against the FP64 oracle.

Tolerances (FP32 kernels vs FP64 oracle, same float32 inputs): total loss
relative error <= 1e-5; gradient error <= 1e-4 normwise per parameter class
(max |g - g_ref| / max |g_ref| over the class).
"""
import dataclasses

import numpy as np
import pytest

import oracle as O
from paper_2604_00250_amd import inputs as I

from gpu_helpers import (LOSS_RTOL, assert_parity, masked_group, merged_grad, oracle_problem, run_gpu, run_oracle, say,
                         theta32, with_theta)

pytestmark = pytest.mark.gpu


def _check_groups(name, groups, launch=None, loss_rtol=1e-5, grad_rtol=1e-4):
    say(f"[{name}] groups={len(groups)} V={[g.n_vox for g in groups]} launch={launch}")
    r = run_gpu(groups, [g.theta for g in groups], launch=launch)
    assert r["status"] == 0, r["status"]
    for i, g in enumerate(groups):
        out, grad, _ = run_oracle(g, g.theta)
        assert_parity(f"{name}/{i}", r["loss"][i], merged_grad(r["gmicro"][i], r["gcal"][i]), out, grad,
                      loss_rtol, grad_rtol)
    return r


@pytest.mark.parametrize("priors", [("rep",), I.PRIOR_NAMES])
@pytest.mark.parametrize("perturb", [False, True])
def test_patch8_n33_mse(priors, perturb):
    w = I.patch8_crossings(priors=priors)
    g = w.groups[0]
    if perturb:
        g = with_theta(g, I.perturb_theta(g.theta, np.random.default_rng(5)))
    _check_groups(f"patch8 priors={len(priors)} perturb={perturb}", [g])


@pytest.mark.parametrize("perturb", [False, True])
def test_patch16_n288_nll_calibrated(perturb):
    g = I.patch16_hcp().groups[0]
    if perturb:
        g = with_theta(g, I.perturb_theta(g.theta, np.random.default_rng(6)))
    _check_groups(f"patch16 nll perturb={perturb}", [g])


def test_phantom_crossing_subpatch_learned_diffusivities():
    w = I.tube_phantom()
    corner = I.crossing_subpatch(w, 4)
    g = I.sub_box(w.groups[0], corner, 4)
    g = with_theta(g, I.perturb_theta(g.theta, np.random.default_rng(7)))
    _check_groups("phantom 4^3 K=4 nll learned-D", [g])


RAGGED = [
    dict(shape=(7, 5, 9), K=2, mode="mse", seed=1, acq_kind="two96", bias="poly2"),
    dict(shape=(6, 6, 6), K=4, mode="nll", seed=2, acq_kind="single33", bias="trilinear8"),
    dict(shape=(9, 4, 11), K=3, mode="mse", seed=3, acq_kind="three288", bias="none", nbh=26),
    dict(shape=(5, 7, 5), K=1, mode="nll", seed=4, acq_kind="two96", bias="poly2", learn=True),
    dict(shape=(3, 3, 3), K=5, mode="mse", seed=5, acq_kind="single33", bias="poly2"),
    dict(shape=(10, 10, 3), K=6, mode="nll", seed=6, acq_kind="two96", bias="none", fill=0.5),
]


@pytest.mark.parametrize("launch", [None, dict(vox_per_lane=1, n_split=1, item_vox=256),
                                    dict(vox_per_lane=1, n_split=4, item_vox=64),
                                    dict(vox_per_lane=2, n_split=1, item_vox=512),
                                    dict(vox_per_lane=2, n_split=2, item_vox=256)])
def test_ragged_masked_mixed_groups(launch):
    groups = [masked_group(**kw) for kw in RAGGED]
    _check_groups("ragged", groups, launch=launch)


@pytest.mark.parametrize("order", ["shells", "interleaved"])
@pytest.mark.parametrize("launch", [None, dict(vox_per_lane=1, n_split=2, item_vox=128)])
def test_mse_acquisition_order(order, launch):
    """The same measurements shell by shell (the b = 0 ones first, which the
    pass takes as whole b = 0 tiles) and in a random order (b = 0 measurements
    scattered through the acquisition, every tile mixing shells), with the
    range also split over two waves."""
    g = masked_group(shape=(11, 9, 7), K=3, mode="mse", seed=21, acq_kind="three288", bias="poly2", fill=0.9)
    if order == "interleaved":
        perm = np.random.default_rng(3).permutation(g.acq.n)
        acq = I.Acquisition(bval=g.acq.bval[perm], bvec=g.acq.bvec[perm], name="three288-interleaved")
        th = dict(g.theta)
        th["alpha"], th["beta"] = th["alpha"][perm], th["beta"][perm]
        g = dataclasses.replace(g, acq=acq, y=np.ascontiguousarray(g.y[perm]), theta=th)
    _check_groups(f"order={order}", [g], launch=launch)


def test_many_items_per_group_and_ragged_tail():
    g = masked_group(shape=(23, 19, 17), K=3, mode="mse", seed=11, acq_kind="three288", bias="poly2", fill=0.8)
    _check_groups("multi-item", [g], launch=dict(vox_per_lane=1, n_split=2, item_vox=128))


def test_empty_group_contributes_only_calibration_prior():
    g0 = masked_group(shape=(4, 4, 4), K=2, mode="mse", seed=8, acq_kind="single33")
    empty = dataclasses.replace(g0, mask=np.zeros((4, 4, 4), dtype=bool), y=np.zeros((33, 0), np.float32),
                                theta={k: (v[..., :0] if k not in ("bias", "alpha", "beta", "sigma_log") else v)
                                       for k, v in g0.theta.items()})
    r = run_gpu([g0, empty], [g0.theta, empty.theta])
    assert r["status"] == 0
    out, _, _ = O.objective(O.Problem(coords=np.zeros((0, 3), dtype=int), shape=(4, 4, 4), bval=g0.acq.bval,
                                      bvec=g0.acq.bvec, K=2, mode="mse", bias="poly2"),
                            theta32(empty.theta), np.zeros((33, 0))), None, None
    assert r["loss"][1][9] == pytest.approx(out["total"], rel=1e-6, abs=1e-12)
    assert r["loss"][1][0] == 0.0
    cal = theta32(empty.theta)
    assert np.allclose(r["gcal"][1]["alpha"], 0.02 * cal["alpha"], rtol=1e-5, atol=1e-9)
    out0, grad0, _ = run_oracle(g0, g0.theta)
    assert_parity("nonempty-beside-empty", r["loss"][0], merged_grad(r["gmicro"][0], r["gcal"][0]), out0, grad0)


@pytest.mark.parametrize("edges", [[(5, 1, 9)], [(17, 17, 17)], [(23, 22, 21)], [(33, 34, 35)],
                                   [(23, 22, 21), (9, 9, 9), (33, 34, 35), (12, 1, 1), (21, 21, 21), (8, 7, 30)]])
@pytest.mark.parametrize("nll", [False, True])
def test_bias_grid_gradient_by_waves_and_by_blocks(edges, nll):
    """Control points of the 8^3 grid whose boxes a wave takes in one round, in several
    (more than four such groups) and whose boxes take a block, one axis a single voxel;
    the fused iteration bit for bit the separate steps."""
    import torch
    from paper_2604_00250_amd.problem import DeviceState, Problem
    rng = np.random.default_rng(len(edges) + edges[0][0])
    acq = I.Acquisition(bval=np.array([0.0, 1.0, 2.0, 2.0]), bvec=I.uniform_sphere(4, rng))
    groups = []
    for e in edges:
        mask = rng.random(e) < 0.9
        g = I.Group(shape=e, mask=mask, acq=acq, K=1, mode="nll" if nll else "mse", bias="trilinear8",
                    priors=("rep", "cal", "tv"))
        g.y = rng.uniform(0.1, 1.0, size=(4, g.n_vox)).astype(np.float32)
        g = with_theta(g, I.perturb_theta(I.init_theta(g.n_vox, 1, 4, 512, rng, sigma_init=0.1), rng, scale=0.2))
        groups.append(g)
    _check_groups(f"grid {edges}", groups)
    states = []
    for fused in (True, False):
        st = DeviceState(Problem(groups), ys=[g.y for g in groups], thetas=[g.theta for g in groups])
        for _ in range(2):
            st.iteration(lr=1e-2) if fused else st.iteration_unfused(lr=1e-2)
        torch.cuda.synchronize()
        states.append(st)
    for a in ("params", "m", "v", "step", "loss"):
        assert torch.equal(getattr(states[0], a), getattr(states[1], a)), a


@pytest.mark.parametrize("n_split", [1, 2, 4])
@pytest.mark.parametrize("K,learn_d", [(2, False), (2, True), (3, False), (6, True)])
def test_rician_items_of_two_voxels_per_lane(K, learn_d, n_split):
    """Rician variants with and without a kernel of two voxels per lane in that launch
    shape: rows of 128 voxels one row of 64 after the other, the last ones short (640 + 65
    voxels), against the oracle and the fused step bit for bit the separate ones."""
    import torch
    from paper_2604_00250_amd.problem import DeviceState, Problem
    rng = np.random.default_rng(10 * K + n_split)
    shape, V, N = (5, 15, 10), 705, 21
    mask = np.zeros(750, dtype=bool)
    mask[:V] = True
    acq = I.Acquisition(bval=np.sort(rng.integers(0, 4, size=N)).astype(np.float64), bvec=I.uniform_sphere(N, rng))
    g = I.Group(shape=shape, mask=mask.reshape(shape), acq=acq, K=K, mode="nll", bias="poly2", learn_diffusivity=learn_d)
    g.y = rng.uniform(0.05, 1.0, size=(N, V)).astype(np.float32)
    g = with_theta(g, I.perturb_theta(I.init_theta(V, K, N, 10, rng, sigma_init=0.1, learn_diffusivity=learn_d), rng,
                                      scale=0.3))
    launch = dict(vox_per_lane=2, n_split=n_split)
    r = _check_groups(f"two per lane K={K} {learn_d} split {n_split}", [g], launch=launch)
    assert r["prob"].plan_info()["items"] == -(-V // (512 // n_split))
    states = []
    for fused in (True, False):
        st = DeviceState(Problem([g], launch=launch), ys=[g.y], thetas=[g.theta])
        for _ in range(2):
            st.iteration(lr=1e-2) if fused else st.iteration_unfused(lr=1e-2)
        torch.cuda.synchronize()
        states.append(st)
    for a in ("params", "m", "v", "step", "loss"):
        assert torch.equal(getattr(states[0], a), getattr(states[1], a)), a


def test_variant_count_does_not_depend_on_the_rows():
    """Two groups of one variant whose N give the split kernel rows of different length are
    two launches but one variant."""
    from paper_2604_00250_amd.problem import Problem
    rng = np.random.default_rng(3)
    mask = np.ones((15, 20, 20), dtype=bool)
    groups = [I.Group(shape=mask.shape, mask=mask, K=1, mode="mse", priors=("rep",),
                      acq=I.Acquisition(bval=np.ones(n), bvec=I.uniform_sphere(n, rng))) for n in (33, 288)]
    prob = Problem(groups)
    assert prob.plan_info()["launches"] == 2
    assert prob.info.n_buckets == 1


@pytest.mark.parametrize("V", [1, 63, 64, 65, 128, 129, 256, 257])
@pytest.mark.parametrize("N", [1, 3, 34])
def test_forward_model_at_the_edges_of_its_rows(V, N):
    """Items of one, two and four rows of 64 voxels, the last row short, with fewer and with
    more measurements than the waves that share a row; nothing written past the last voxel."""
    import torch
    from paper_2604_00250_amd.problem import DeviceState, Problem
    rng = np.random.default_rng(V + 1000 * N)
    shape = (2, -(-V // 20), 10)
    mask = np.zeros(20 * shape[1], dtype=bool)
    mask[:V] = True
    acq = I.Acquisition(bval=rng.integers(0, 4, size=N).astype(np.float64), bvec=I.uniform_sphere(N, rng))
    g = I.Group(shape=shape, mask=mask.reshape(shape), acq=acq, K=2, mode="mse", bias="poly2")
    g.theta = I.perturb_theta(I.init_theta(V, 2, N, 10, rng), rng, scale=0.3)
    prob = Problem([g], launch=dict(vox_per_lane=1, n_split=1))
    st = DeviceState(prob, thetas=[g.theta])
    out = torch.full((st.n_y + 64,), -7.0, device=st.device)
    st.synthesize(out)
    torch.cuda.synchronize()
    ref = O.synthesize(oracle_problem(g), theta32(g.theta))
    got = out[:st.n_y].cpu().numpy().reshape(N, V)
    assert np.abs(got - ref).max() < 2e-6 * np.abs(ref).max()
    assert bool((out[st.n_y:] == -7.0).all())


@pytest.mark.parametrize("n_split,N", [(4, 31), (4, 32), (2, 15), (2, 16)])
def test_forward_model_of_many_short_items(n_split, N):
    """More blocks than fill the device, of one or two rows: waves share a row from eight
    measurements each up, else take one each."""
    import torch
    from paper_2604_00250_amd.problem import DeviceState, Problem
    rng = np.random.default_rng(N)
    rows = 256 // n_split
    V = rows * 1025 + rows - 9
    shape = (10, -(-V // 1000), 100)
    mask = np.zeros(1000 * shape[1], dtype=bool)
    mask[:V] = True
    acq = I.Acquisition(bval=rng.integers(0, 4, size=N).astype(np.float64), bvec=I.uniform_sphere(N, rng))
    g = I.Group(shape=shape, mask=mask.reshape(shape), acq=acq, K=1, mode="mse")
    g.theta = I.perturb_theta(I.init_theta(V, 1, N, 0, rng), rng, scale=0.3)
    prob = Problem([g], launch=dict(vox_per_lane=1, n_split=n_split))
    assert prob.plan_info()["items"] == 1026
    st = DeviceState(prob, thetas=[g.theta])
    out = torch.full((st.n_y,), -7.0, device=st.device)
    st.synthesize(out)
    torch.cuda.synchronize()
    ref = O.synthesize(oracle_problem(g), theta32(g.theta))
    assert np.abs(out.cpu().numpy().reshape(N, V) - ref).max() < 2e-6 * np.abs(ref).max()


def test_synthesize_matches_oracle_forward():
    import torch
    from paper_2604_00250_amd.problem import DeviceState, Problem
    groups = [masked_group(**kw) for kw in RAGGED[:4]]
    prob = Problem(groups)
    st = DeviceState(prob, ys=[g.y for g in groups], thetas=[g.theta for g in groups])
    out = st.synthesize()
    torch.cuda.synchronize()
    yh = prob.unpack_y(out.cpu().numpy())
    for g, a in zip(groups, yh):
        ref = O.synthesize(O.Problem(coords=g.coords, shape=g.shape, bval=g.acq.bval, bvec=g.acq.bvec, K=g.K,
                                     mode=g.mode, bias=g.bias, learn_diffusivity=g.learn_diffusivity),
                           theta32(g.theta))
        err = np.abs(a - ref).max() / np.abs(ref).max()
        say(f"[synth] K={g.K} max rel err {err:.2e}")
        assert err < 2e-6


def test_adam_and_rprop_match_oracle_elementwise():
    import torch
    from paper_2604_00250_amd.problem import adam_step_ptr, rprop_step_ptr
    rng = np.random.default_rng(0)
    n = 100_003
    p0 = rng.normal(0, 1, n).astype(np.float32)
    dev = torch.device("cuda:0")
    p = torch.from_numpy(p0.copy()).to(dev)
    m = torch.zeros(n, device=dev)
    v = torch.zeros(n, device=dev)
    step = torch.zeros(2, dtype=torch.int32, device=dev)
    pr, mr, vr = p0.astype(np.float64), np.zeros(n), np.zeros(n)
    s = torch.cuda.current_stream().cuda_stream
    for t in range(1, 6):
        g = rng.normal(0, 1, n).astype(np.float32)
        gt = torch.from_numpy(g).to(dev)
        adam_step_ptr(p.data_ptr(), gt.data_ptr(), m.data_ptr(), v.data_ptr(), n, 1e-2, 0.9, 0.999, 1e-8,
                      step.data_ptr(), s)
        pr, mr, vr = O.adam_step(pr, g.astype(np.float64), mr, vr, t)
    torch.cuda.synchronize()
    assert step.cpu().tolist() == [5, 0]
    assert np.abs(p.cpu().numpy() - pr).max() < 1e-5
    # Rprop
    p = torch.from_numpy(p0.copy()).to(dev)
    prev = torch.zeros(n, device=dev)
    st = torch.full((n,), 0.01, device=dev)
    pr, prevr, str_ = p0.astype(np.float64), np.zeros(n), np.full(n, 0.01)
    for t in range(6):
        g = rng.normal(0, 1, n).astype(np.float32)
        g[::7] = 0.0
        gt = torch.from_numpy(g).to(dev)
        rprop_step_ptr(p.data_ptr(), gt.data_ptr(), prev.data_ptr(), st.data_ptr(), n, 0.5, 1.2, 1e-6, 50.0, s)
        pr, prevr, str_ = O.rprop_step(pr, g, prevr, str_)
    torch.cuda.synchronize()
    assert np.abs(st.cpu().numpy() - str_).max() < 1e-7
    assert np.abs(p.cpu().numpy() - pr).max() < 1e-6


def test_bitwise_determinism_and_direction_sign_invariance():
    groups = [masked_group(**kw) for kw in RAGGED[:3]]
    r1 = run_gpu(groups, [g.theta for g in groups])
    r2 = run_gpu(groups, [g.theta for g in groups], repeat=2)
    assert np.array_equal(r1["loss"], r2["loss"])
    for a, b in zip(r1["gmicro"], r2["gmicro"]):
        for k in a:
            assert np.array_equal(a[k], b[k]), k
    flipped = []
    for g in groups:
        th = dict(g.theta)
        th["v"] = -th["v"]
        flipped.append(th)
    r3 = run_gpu(groups, flipped)
    assert np.array_equal(r1["loss"], r3["loss"])
    for a, b in zip(r1["gmicro"], r3["gmicro"]):
        assert np.array_equal(a["v"], -b["v"])


def test_status_bits_for_zero_direction_and_nonfinite_data():
    g = masked_group(shape=(4, 4, 4), K=2, mode="mse", seed=9, acq_kind="single33")
    th = {k: v.copy() for k, v in g.theta.items()}
    th["v"][1, :, 5] = 0.0
    r = run_gpu([g], [th])
    assert r["status"] & 4
    y = g.y.copy()
    y[3, 7] = np.nan
    r = run_gpu([dataclasses.replace(g, y=y)], [g.theta])
    assert r["status"] & 1 and r["status"] & 2
    # NLL with an infinite noise level: the loss is not finite
    gn = masked_group(shape=(4, 4, 4), K=2, mode="nll", seed=10, acq_kind="single33")
    th = {k: v.copy() for k, v in gn.theta.items()}
    th["sigma_log"] = np.array(np.inf, dtype=np.float32)
    r = run_gpu([gn], [th])
    assert r["status"] & 1
    th["sigma_log"] = np.array(-np.inf, dtype=np.float32)
    r = run_gpu([gn], [th])
    assert r["status"] & 1


def test_workspace_smaller_than_required_is_rejected():
    import ctypes
    import torch
    from paper_2604_00250_amd import _lib as L
    g = masked_group(shape=(5, 4, 3), K=2, mode="mse", seed=12, acq_kind="single33")
    r = run_gpu([g], [g.theta])
    st = r["state"]
    need = st.prob.workspace_bytes()
    assert need > 0
    pm, pc, gm, gc = st.ptrs()
    rc = L.lib().prism_loss_grad(st.prob.handle, st.y.data_ptr(), pm, pc, st.loss.data_ptr(), gm, gc,
                                 st.ws.data_ptr(), need - 1, st.status.data_ptr(), None)
    assert rc == L.PRISM_E_WORKSPACE
    assert "workspace" in L.lib().prism_last_error().decode()
    rc = L.lib().prism_loss_grad(st.prob.handle, st.y.data_ptr(), pm, pc, st.loss.data_ptr(), gm, gc,
                                 None, need, st.status.data_ptr(), None)
    assert rc == L.PRISM_E_INVALID
    torch.cuda.synchronize()


def test_only_the_iteration_needs_the_copy_of_the_directions():
    """A continuity problem's gradient call takes a workspace without it, with the same
    bits and nothing written past its end; one byte less is refused, and so is the
    iteration."""
    import torch
    from paper_2604_00250_amd import _lib as L
    g = masked_group(shape=(7, 6, 5), K=3, mode="mse", seed=13, acq_kind="single33", priors=("spatial", "continuity"))
    r = run_gpu([g], [g.theta])
    st = r["state"]
    full = st.prob.workspace_bytes()
    need = full - -(-12 * 3 * g.n_vox // 256) * 256
    loss, grad = st.loss.clone(), st.grad.clone()
    st.ws.fill_(0xA5)
    st.loss.zero_()
    st.grad.zero_()
    pm, pc, gm, gc = st.ptrs()

    def call(n):
        return L.lib().prism_loss_grad(st.prob.handle, st.y.data_ptr(), pm, pc, st.loss.data_ptr(), gm, gc,
                                       st.ws.data_ptr(), n, st.status.data_ptr(), st._s())
    assert call(need - 1) == L.PRISM_E_WORKSPACE
    assert call(need) == 0
    torch.cuda.synchronize()
    assert torch.equal(st.loss, loss) and torch.equal(st.grad, grad)
    assert bool((st.ws[need:full] == 0xA5).all())
    st.ws_bytes = full - 1
    with pytest.raises(L.PrismError):
        st.iteration(lr=1e-2)


@pytest.mark.parametrize("n_items", [1, 32, 33, 256, 257, 1500, 1501])
def test_record_reduction_at_the_edges_of_its_tiles(n_items):
    """Items of 64 voxels, the last one short: the reduction's wide and narrow tiles,
    its two block sizes and the runs summed first, against the oracle."""
    V = 64 * n_items - 5
    shape = (5, -(-V // 500), 100)
    mask = np.zeros(5 * shape[1] * 100, dtype=bool)
    mask[:V] = True
    rng = np.random.default_rng(n_items)
    bval = np.array([0.0, 0.0, 1.0, 1.0, 2.0, 2.0, 3.0])
    acq = I.Acquisition(bval=bval, bvec=I.uniform_sphere(bval.size, rng))
    g = I.Group(shape=shape, mask=mask.reshape(shape), acq=acq, K=1, mode="mse", bias="poly2", neighbourhood=0,
                priors=("rep", "sparse", "cal"))
    g.y = rng.uniform(0.1, 1.0, size=(acq.n, V)).astype(np.float32)
    g = with_theta(g, I.perturb_theta(I.init_theta(V, 1, acq.n, 10, rng), rng))
    r = _check_groups(f"{n_items} items", [g], launch=dict(vox_per_lane=1, n_split=4, item_vox=64))
    assert r["prob"].plan_info()["items"] == n_items


@pytest.mark.parametrize("n_items", [32, 33, 257, 1501])
def test_rician_loss_of_the_fused_iteration_is_at_the_sigma_before_it(n_items):
    """Up to 32 items one block of the reduction has both the loss and sigma's update;
    above they are in two.  Loss rows, history and every updated value are those of the
    gradient call and the separate Adam step, bit for bit, and the first loss the oracle's
    at the parameters before the step (the step moves the loss by more than 100 times the
    bound)."""
    import torch
    from paper_2604_00250_amd.problem import DeviceState, Problem
    V = 64 * n_items - 5
    shape = (5, -(-V // 500), 100)
    mask = np.zeros(5 * shape[1] * 100, dtype=bool)
    mask[:V] = True
    rng = np.random.default_rng(n_items)
    bval = np.array([0.0, 0.0, 1.0, 1.0, 2.0, 2.0, 3.0])
    acq = I.Acquisition(bval=bval, bvec=I.uniform_sphere(bval.size, rng))
    g = I.Group(shape=shape, mask=mask.reshape(shape), acq=acq, K=1, mode="nll", bias="poly2", neighbourhood=0,
                priors=("rep", "sparse", "cal"))
    g.y = rng.uniform(0.1, 1.0, size=(acq.n, V)).astype(np.float32)
    g = with_theta(g, I.perturb_theta(I.init_theta(V, 1, acq.n, 10, rng, sigma_init=0.1), rng))
    states = []
    for fused in (True, False):
        prob = Problem([g], launch=dict(vox_per_lane=1, n_split=4, item_vox=64))
        st = DeviceState(prob, ys=[g.y], thetas=[g.theta])
        hist = torch.zeros((2, 1, len(O.TERMS)), dtype=torch.float64, device=st.device)
        rows = []
        for _ in range(2):
            st.iteration(lr=1e-2, history=hist) if fused else st.iteration_unfused(lr=1e-2)
            torch.cuda.synchronize()
            rows.append(st.loss.clone())
        states.append((st, rows, hist))
    (a, rows_a, hist), (b, rows_b, _) = states
    assert a.prob.plan_info()["items"] == n_items
    for t in range(2):
        assert torch.equal(rows_a[t], rows_b[t]) and torch.equal(hist[t], rows_a[t]), t
    for name in ("params", "m", "v", "step"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
    out, _, _ = run_oracle(g, g.theta)
    it = O.TERMS.index("total")
    got = float(rows_a[0][0, it])
    assert abs(got - out["total"]) <= LOSS_RTOL * abs(out["total"])
    assert 2e-2 * acq.n * V > 100 * LOSS_RTOL * abs(out["total"])


@pytest.mark.parametrize("V,N", [(1, 1), (15, 3), (16, 17), (17, 33), (4095, 7), (4097, 31), (8190, 16), (8193, 40),
                                 (16386, 5)])
@pytest.mark.parametrize("K,mode,learn_d", [(1, "mse", False), (3, "nll", False), (2, "mse", True), (6, "nll", True)])
def test_small_problems_in_rows_of_16_32_and_64_voxels(V, N, K, mode, learn_d):
    """The split kernels at the ends of their ranges: fewer measurements than slots and
    ragged shares, short last rows, both sides of each change of row length; gradient
    against the oracle and the fused Adam step bit for bit the unfused one's."""
    import torch
    from paper_2604_00250_amd.problem import DeviceState, Problem
    rng = np.random.default_rng(V + 100 * N + K)
    shape = (3, -(-V // 60), 20)
    mask = np.zeros(60 * shape[1], dtype=bool)
    mask[:V] = True
    bval = np.sort(rng.integers(0, 4, size=N)).astype(np.float64)
    bval[-1] = max(bval[-1], 1.0)   # at b = 0 alone the data term has no gradient in the fractions
    acq = I.Acquisition(bval=bval, bvec=I.uniform_sphere(N, rng))
    g = I.Group(shape=shape, mask=mask.reshape(shape), acq=acq, K=K, mode=mode, bias="poly2", learn_diffusivity=learn_d,
                neighbourhood=6)
    g.y = rng.uniform(0.05, 1.0, size=(N, V)).astype(np.float32)
    g = with_theta(g, I.perturb_theta(I.init_theta(V, K, N, 10, rng, sigma_init=0.1 if mode == "nll" else 0.0,
                                                   learn_diffusivity=learn_d), rng, scale=0.3))
    _check_groups(f"V={V} N={N} K={K} {mode}", [g])
    states = []
    for fused in (True, False):
        prob = Problem([g])
        st = DeviceState(prob, ys=[g.y], thetas=[g.theta])
        for _ in range(2):
            st.iteration(lr=1e-2) if fused else st.iteration_unfused(lr=1e-2)
        torch.cuda.synchronize()
        states.append(st)
    for a in ("params", "m", "v", "step", "loss"):
        assert torch.equal(getattr(states[0], a), getattr(states[1], a)), a


@pytest.mark.parametrize("V,N,K,mode,learn_d", [(32769, 7, 4, "nll", True), (61000, 5, 4, "nll", True),
                                                (61000, 9, 2, "nll", False), (49153, 6, 5, "nll", False)])
def test_rows_of_64_voxels_in_two_rounds(V, N, K, mode, learn_d):
    """Problems whose rows of 64 are more blocks than the device holds at once, where the
    fused pass would need two rounds as well (the shortest is one past a full round)."""
    test_small_problems_in_rows_of_16_32_and_64_voxels(V, N, K, mode, learn_d)


@pytest.mark.parametrize("order", ["sorted", "interleaved", "all_different", "one_b", "b0_only_groups"])
@pytest.mark.parametrize("N,mode,learn_d,launch", [(3, "mse", False, None), (41, "nll", True, dict(vox_per_lane=2, n_split=1)),
                                                   (50, "mse", False, dict(vox_per_lane=1, n_split=2)),
                                                   (64, "mse", True, dict(vox_per_lane=1, n_split=1, item_vox=512)),
                                                   (30, "nll", False, dict(vox_per_lane=1, n_split=4, item_vox=64))])
def test_runs_of_equal_b_in_any_order_of_the_acquisition(order, N, mode, learn_d, launch):
    """Runs, left-over measurements and partial groups, taken in the library's own order
    and returned in the caller's: every launch shape that has the measurement loop."""
    rng = np.random.default_rng(N)
    b = np.array([0.0, 1.0, 2.0, 3.0])[rng.integers(0, 4, size=N)]
    b[0] = 1.0
    if order == "sorted":
        b = np.sort(b)
    elif order == "all_different":
        b = 0.5 + np.arange(N) / N
    elif order == "one_b":
        b[:] = 2.0
    elif order == "b0_only_groups":
        b = np.where(np.arange(N) % 9 < 8, 0.0, 0.5 + np.arange(N) / N)
        b[0] = 1.0
    acq = I.Acquisition(bval=b, bvec=I.uniform_sphere(N, rng))
    shape = (5, 7, 19)
    mask = rng.random(shape) < 0.9
    V = int(mask.sum())
    g = I.Group(shape=shape, mask=mask, acq=acq, K=3, mode=mode, bias="poly2", learn_diffusivity=learn_d)
    g.y = rng.uniform(0.05, 1.0, size=(N, V)).astype(np.float32)
    g = with_theta(g, I.perturb_theta(I.init_theta(V, 3, N, 10, rng, sigma_init=0.1 if mode == "nll" else 0.0,
                                                   learn_diffusivity=learn_d), rng, scale=0.3))
    _check_groups(f"{order} N={N} {mode} {launch}", [g], launch=launch)
