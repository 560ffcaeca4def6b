"""prism_loss_grad_noalloc (the entry point whose workspace is the library's
static device array) against prism_loss_grad (caller workspace): bit for bit
on two calls in a row, the second on a smaller problem, so the second call
runs on what the first left in the shared array; and a problem whose
workspace exceeds the static array is refused before anything is queued."""
import ctypes

import numpy as np
import pytest

from paper_2604_00250_amd import _lib as L
from paper_2604_00250_amd import inputs as I

from gpu_helpers import say

pytestmark = pytest.mark.gpu


def _compare(group, theta):
    import torch
    from paper_2604_00250_amd.problem import DeviceState, Problem
    prob = Problem([group])
    st = DeviceState(prob, ys=[group.y], thetas=[theta])
    st.loss_grad()
    torch.cuda.synchronize()
    loss_ref, grad_ref, status_ref = st.loss.clone(), st.grad.clone(), st.status.clone()
    loss = torch.full_like(st.loss, float("nan"))
    grad = torch.full_like(st.grad, float("nan"))
    status = torch.zeros_like(st.status)
    pm, pc, _, _ = st.ptrs()
    gm = grad.data_ptr()
    prob.loss_grad_noalloc_ptr(st.y.data_ptr(), pm, pc, loss.data_ptr(), gm, gm + 4 * st.n_micro,
                               status.data_ptr(), st._s())
    torch.cuda.synchronize()
    say(f"[noalloc] V={group.n_vox} N={group.acq.n} workspace {prob.workspace_bytes()} B "
        f"loss {loss[0, -1].item():.10g} ref {loss_ref[0, -1].item():.10g}")
    assert int(status_ref.item()) == 0
    assert torch.equal(loss, loss_ref)
    assert torch.equal(grad, grad_ref)
    assert torch.equal(status, status_ref)


def test_noalloc_is_bitwise_loss_grad_on_two_calls_in_a_row():
    large = I.patch16_hcp().groups[0]            # 4096 voxels, N = 288, NLL, calibration
    small = I.patch8_crossings(priors=I.PRIOR_NAMES).groups[0]   # 512 voxels, N = 33
    _compare(large, I.perturb_theta(large.theta, np.random.default_rng(5), scale=0.5))
    _compare(small, I.perturb_theta(small.theta, np.random.default_rng(6), scale=0.5))


def test_noalloc_refuses_a_problem_beyond_the_static_workspace():
    import torch
    from paper_2604_00250_amd.problem import Problem
    acq = I.Acquisition(bval=np.zeros(1), bvec=np.array([[1.0, 0.0, 0.0]]))
    shape = (200, 200, 100)   # 4M voxels with the Eq. 7 prior: ~128 MB of [V][cs] rows
    g = I.Group(shape=shape, mask=np.ones(shape, dtype=bool), acq=acq, K=1, mode="mse",
                priors=("spatial",))
    prob = Problem([g])
    need = prob.workspace_bytes()
    assert need > L.NOALLOC_WORKSPACE_BYTES
    buf = torch.zeros(16, dtype=torch.float64, device="cuda:0")
    p = buf.data_ptr()
    rc = L.lib().prism_loss_grad_noalloc(prob.handle, p, p, p, p, p, p, p, None)
    msg = L.lib().prism_last_error().decode()
    say(f"[noalloc] workspace {need} B: rc {rc}: {msg}")
    assert rc == L.PRISM_E_WORKSPACE and "static workspace" in msg
    torch.cuda.synchronize()
    assert not torch.any(buf)  # nothing was queued


@pytest.mark.parametrize("n_groups,fits", [(700, True), (800, False)])
def test_finer_items_neither_cost_nor_gain_the_static_workspace(n_groups, fits):
    """Groups of 256 voxels, N = 1024, in the automatic cut: 700 of them fit the static
    workspace as one item each (49.3 MiB) but not as four (82.5), so they run, bit for bit
    as with a caller's workspace; 800 never fitted (69 MiB with the partial sums that the
    coarser cut was reduced through) and are refused."""
    import torch
    from paper_2604_00250_amd.problem import DeviceState, Problem
    rng = np.random.default_rng(n_groups)
    b = np.full(1024, 2.0)
    b[::9] = 0.0
    acq = I.Acquisition(bval=b, bvec=I.uniform_sphere(1024, rng))
    shape = (16, 16, 1)
    groups = [I.Group(shape=shape, mask=np.ones(shape, dtype=bool), acq=acq, K=1, mode="mse", priors=("spatial",))
              for _ in range(n_groups)]
    prob = Problem(groups)
    say(f"[noalloc] {n_groups} groups: workspace {prob.workspace_bytes()} B, plan {prob.plan_info()}")
    assert (prob.workspace_bytes() <= L.NOALLOC_WORKSPACE_BYTES) == fits
    st = DeviceState(prob)
    st.params[:st.n_micro].normal_()
    st.y.uniform_(0.1, 1.0)
    pm, pc, gm, gc = st.ptrs()
    loss, grad, status = torch.zeros_like(st.loss), torch.zeros_like(st.grad), torch.zeros_like(st.status)
    rc = L.lib().prism_loss_grad_noalloc(prob.handle, st.y.data_ptr(), pm, pc, loss.data_ptr(), grad.data_ptr(),
                                         grad.data_ptr() + 4 * st.n_micro, status.data_ptr(), st._s())
    assert rc == (0 if fits else L.PRISM_E_WORKSPACE), L.lib().prism_last_error().decode()
    torch.cuda.synchronize()
    if fits:
        st.loss_grad()
        torch.cuda.synchronize()
        assert torch.equal(loss, st.loss) and torch.equal(grad, st.grad)
        assert int(status.item()) == 0 and float(loss[:, -1].min()) > 0.0
    else:
        assert not torch.any(loss) and not torch.any(grad)
