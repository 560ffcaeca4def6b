"""Eq. 9 on the GPU: the device's special functions against SciPy over
float32 arguments in [0, 1e5] (the 2e-7 relative bound), and parity of the
Rician NLL pass with the oracle where z = |y| |yhat| / sigma^2 reaches 1e4
(high SNR) and where every z is below the branch split (low SNR)."""
import importlib.util
import math
import os

import numpy as np
import pytest

import oracle as O

from gpu_helpers import assert_parity, masked_group, merged_grad, run_gpu, run_oracle, say, theta32, oracle_problem

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))


def _gen():
    spec = importlib.util.spec_from_file_location(
        "gen_bessel_fit", os.path.join(HERE, "..", "paper_2604_00250_amd", "csrc", "gen_bessel_fit.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_device_special_functions_meet_the_bound():
    import torch
    from paper_2604_00250_amd import _lib as L
    gen = _gen()
    z = gen.test_grid()
    dev = torch.from_numpy(z).cuda()
    out = [torch.empty_like(dev) for _ in range(3)]
    L.check(L.lib().prism_rician_terms(dev.data_ptr(), out[0].data_ptr(), out[1].data_ptr(), out[2].data_ptr(),
                                       z.size, None))
    torch.cuda.synchronize()
    vals = [o.cpu().numpy() for o in out]
    errs = gen.relative_errors(z, vals)
    emu = gen.evaluate_f32(z)
    ulps = [float(np.max(np.abs(a.astype(np.float64) - b) / np.spacing(np.abs(b).astype(np.float32)).astype(np.float64)))
            for a, b in zip(vals, emu)]
    say(f"[bessel] {z.size} arguments: max relative error log I0e {errs[0].max():.3e} (z={z[errs[0].argmax()]:.6g}), "
        f"1-R {errs[1].max():.3e} (z={z[errs[1].argmax()]:.6g}), q {errs[2].max():.3e}; "
        f"device vs host emulation within {ulps} ulp")
    for e in errs:
        assert e.max() <= 2e-7


def test_device_small_arguments_and_q_take_one_rounding():
    """The two results whose only error of note is one rounding, 2^-24: log I0e on
    [1e-4, 1/8) within 1.1 of it and q on (0, 65536) within 1.25 (what adds to it is a
    rounding or two of a term at most z/4, respectively a tenth, of the result)."""
    import torch
    from paper_2604_00250_amd import _lib as L
    gen = _gen()
    z = gen.test_grid()
    z = z[(z > 0) & (z < np.float32(65536.0))]
    dev = torch.from_numpy(z).cuda()
    out = [torch.empty_like(dev) for _ in range(3)]
    L.check(L.lib().prism_rician_terms(dev.data_ptr(), out[0].data_ptr(), out[1].data_ptr(), out[2].data_ptr(),
                                       z.size, None))
    torch.cuda.synchronize()
    e_li, _, e_q = gen.relative_errors(z, [o.cpu().numpy() for o in out])
    small = (z >= np.float32(1e-4)) & (z < np.float32(0.125))
    say(f"[bessel] log I0e on [1e-4, 1/8) {e_li[small].max():.3e}, q on (0, 65536) {e_q.max():.3e}")
    assert e_li[small].max() <= 1.1 * 2.0 ** -24
    assert e_q.max() <= 1.25 * 2.0 ** -24


@pytest.mark.parametrize("z", [[0.125, 0.12499999], [65535.996, 65536.0, 65536.01], [1e6, 1e12, 1e30, 1e37], [0.0]])
def test_device_special_functions_at_the_ends_of_the_table_and_beyond(z):
    """Both sides of the table's first interval and of its end, and arguments far
    past the range of a fit (to where 1 - R is still a normal float32): SciPy's i0e / i1e lose 1 - R beyond 1e5, where the
    large-argument expansions are exact to float32.  The bound is that of the
    sweep above."""
    import torch
    from paper_2604_00250_amd import _lib as L
    dev = torch.tensor(z, dtype=torch.float32).cuda()
    out = [torch.empty_like(dev) for _ in range(3)]
    L.check(L.lib().prism_rician_terms(dev.data_ptr(), out[0].data_ptr(), out[1].data_ptr(), out[2].data_ptr(),
                                       len(z), None))
    torch.cuda.synchronize()
    zd = dev.cpu().numpy().astype(np.float64)
    if zd.max() >= 1e5:
        w = 1.0 / zd
        ref = (-0.5 * np.log(2.0 * np.pi * zd) + w / 8, 0.5 * w * (1 + w / 4), 1 + w / 4)
    else:
        ref = _gen().reference(zd)
    for got, want in zip(out, ref):
        got = got.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - want) <= 2e-7 * np.abs(want)), (got, want)


def _z_range(g, th):
    prob = oracle_problem(g)
    yhat = O.synthesize(prob, theta32(th))
    s2 = math.exp(2.0 * float(th["sigma_log"]))
    z = np.abs(np.asarray(g.y, np.float64)) * np.abs(yhat) / s2
    return z


@pytest.mark.parametrize("K,acq", [(3, "three288"), (2, "two96")])
def test_nll_parity_at_high_snr(K, acq):
    g = masked_group((7, 6, 5), K=K, mode="nll", seed=91 + K, acq_kind=acq, snr=100.0)
    th = dict(g.theta)
    th["sigma_log"] = np.float32(math.log(0.01))
    z = _z_range(g, th)
    say(f"[nll high snr] K={K} N={g.acq.n} z in [{z.min():.3g}, {z.max():.3g}], "
        f"{(z >= 3.75).mean() * 100:.0f}% above the split")
    assert z.max() > 1e3
    r = run_gpu([g], [th])
    out, grad, _ = run_oracle(g, th)
    assert r["status"] == 0
    assert_parity(f"nll-high-snr K={K}", r["loss"][0], merged_grad(r["gmicro"][0], r["gcal"][0]), out, grad)


def test_nll_parity_with_every_z_below_the_split():
    g = masked_group((6, 6, 6), K=3, mode="nll", seed=97, acq_kind="three288", snr=3.0)
    th = dict(g.theta)
    th["sigma_log"] = np.float32(0.0)
    z = _z_range(g, th)
    # sigma such that the largest argument sits at 3.0
    th["sigma_log"] = np.float32(0.5 * math.log(z.max() / 3.0))
    z = _z_range(g, th)
    say(f"[nll low z] z in [{z.min():.3g}, {z.max():.3g}]")
    assert z.max() < 3.75
    r = run_gpu([g], [th])
    out, grad, _ = run_oracle(g, th)
    assert r["status"] == 0
    assert_parity("nll-low-z", r["loss"][0], merged_grad(r["gmicro"][0], r["gcal"][0]), out, grad)
