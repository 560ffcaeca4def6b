"""Generate bessel_fit.h: the coefficient table of the Rician NLL (Eq. 9).

The kernels need, for z >= 0,
    log I0e(z) = log I0(z) - z          (the cancellation-free NLL term)
    1 - R(z),  R = I1 / I0              (the NLL adjoint)
    q(z) = 2 z (1 - R(z))               (the d/dsigma_log term)

1 - R is the derivative of -log I0e, so one polynomial per interval of z gives
both: with delta = z - z0,
    -log I0e(z) = c0 + delta (c1 + delta s),   s = c2 + c3 delta + ... + c6 delta^4
    1 - R(z)    = c1 + delta (2 s + delta s')
(the derivative of the first line).  The intervals are [0, 1/8) and the eighths
of every octave from 1/8 up to Z_SPLIT, so the interval of an argument is a
shift of its float32 bits and |delta| <= z/16: the correction to c1 is small and
1 - R keeps the accuracy of c1, of delta (z - z0 is exact: the two lie within a
factor of two) and of one rounding.  On [0, 1/8) (z0 = 0, c0 = 0, c1 = 1)
-log I0e is summed as z + z (z s): in c1 + z s and its product with z both
roundings would count.  c1 .. c6 come from a weighted least squares
fit of 1 - R; z0 is chosen among the float32 numbers near the interval's middle
so that both c0 and c1 are float32 numbers to about a thousandth of an ulp
(accurate tables), which leaves the final rounding as the main error.

From Z_SPLIT up, the large-argument expansions
    log I0e(z) = -log(2 pi z)/2 + 1/(8z),   2 z (1 - R) = 1 + 1/(4z)
whose next terms are below 1e-10 relative there.

`evaluate_f32` below is the kernels' algorithm step by step in float32
arithmetic on the host (hardware reciprocal and log2 modelled as correctly
rounded float32), used by the tests to bound the error against SciPy's float64
i0e / i1e.  Run from the repository root to regenerate:
    python paper_2604_00250_amd/csrc/gen_bessel_fit.py
"""
import os

import numpy as np
from scipy.special import i0e, i1e

f32 = np.float32
Z_FIRST = 0.125        # end of the first interval
Z_SPLIT = 65536.0      # the expansions from here up
SUB_BITS = 3           # mantissa bits that pick the interval within an octave
DEG = 6                # degree of -log I0e's polynomial
SHIFT = 23 - SUB_BITS
HALF_LOG_2PI = 0.5 * np.log(2.0 * np.pi)
HALF_LN2 = 0.5 * np.log(2.0)


def _bits(x):
    return int(np.array(x, f32).view(np.uint32))


BITS_LO = _bits(Z_FIRST) - (1 << SHIFT)      # idx = (clamp(bits) - BITS_LO) >> SHIFT
BITS_HI = _bits(Z_SPLIT) - 1
N_ENTRY = ((BITS_HI - BITS_LO) >> SHIFT) + 1


def targets(z):
    """-log I0e(z) and 1 - R(z) in float64."""
    z = np.asarray(z, dtype=np.float64)
    e0, e1 = i0e(z), i1e(z)
    return -np.log(e0), (e0 - e1) / e0


def interval(i):
    """[lo, hi) of table entry i."""
    if i == 0:
        return 0.0, Z_FIRST
    lo = np.array(BITS_LO + (i << SHIFT), np.uint32).view(f32)
    hi = np.array(BITS_LO + ((i + 1) << SHIFT), np.uint32).view(f32)
    return float(lo), float(hi)


def entry(i):
    """(z0, c0 .. c6) of entry i, float32 values."""
    lo, hi = interval(i)
    if i == 0:
        z0, c0, c1 = 0.0, 0.0, 1.0
    else:
        # float32 candidates over the middle quarter of the interval
        a, b = _bits(lo + 0.375 * (hi - lo)), _bits(lo + 0.625 * (hi - lo))
        cand = np.arange(a, b, dtype=np.uint32).view(f32).astype(np.float64)
        v0, v1 = targets(cand)
        off = np.maximum(np.abs(v0.astype(f32) / v0 - 1.0), np.abs(v1.astype(f32) / v1 - 1.0))
        j = int(off.argmin())
        z0, c0, c1 = cand[j], v0[j], v1[j]
    c1 = float(f32(c1))
    n = 96
    x = -np.cos(np.pi * (np.arange(n) + 0.5) / n)
    z = 0.5 * (lo + hi) + 0.5 * (hi - lo) * x
    h = 0.5 * (hi - lo)
    d = (z - z0) / h
    _, omr = targets(z)
    A = np.stack([d ** k for k in range(1, DEG)], 1) / omr[:, None]
    a, *_ = np.linalg.lstsq(A, (omr - c1) / omr, rcond=None)
    c = [c0, c1] + [a[k - 1] / h ** k / (k + 1) for k in range(1, DEG)]
    return [float(f32(v)) for v in [z0] + c]


def fits():
    """The table [8][N_ENTRY]: z0, c0 .. c6 per interval."""
    return np.array([entry(i) for i in range(N_ENTRY)]).T


# ----------------------------------------------------------------------------
# host emulation of the kernels' evaluation
# ----------------------------------------------------------------------------

def _fma32(a, b, c):
    # the product of two float32 values is exact in float64; one rounding to float32
    return f32(np.float64(a) * np.float64(b) + np.float64(c))


def _rcp32(x):
    return f32(1.0 / np.asarray(x, np.float64))                  # v_rcp_f32


def evaluate_f32(z, table=None):
    """(log I0e(z), 1 - R(z), q(z)) for float32 z >= 0, as the kernels compute them."""
    tab = (fits() if table is None else table).astype(f32)
    z = np.asarray(z, dtype=f32)
    bits = z.view(np.int32).astype(np.int64)
    idx = (np.clip(bits, BITS_LO, BITS_HI) - BITS_LO) >> SHIFT
    z0, c = tab[0][idx], [t[idx] for t in tab[1:]]
    d = f32(z - z0)
    s, ds = c[DEG], c[DEG]
    s = _fma32(s, d, c[DEG - 1])
    for k in range(DEG - 2, 1, -1):
        ds = _fma32(ds, d, s)
        s = _fma32(s, d, c[k])
    t = _fma32(d, ds, f32(s + s))
    omr = _fma32(d, t, c[1])
    nli = _fma32(d, _fma32(d, s, c[1]), c[0])
    nli = np.where(bits < _bits(Z_FIRST) - 1, _fma32(f32(z * s), z, z), nli)
    # q = 2 z (1 - R) from 1 - R and what its rounding left
    z2 = f32(z + z)
    q = _fma32(z2, omr, f32(z2 * _fma32(d, t, f32(c[1] - omr))))
    # from the split up
    big = z >= f32(Z_SPLIT)
    zl = np.where(big, z, f32(1.0))
    iz0 = _rcp32(zl)
    iz = _fma32(_fma32(-zl, iz0, f32(1.0)), iz0, iz0)              # one Newton step
    e = f32(f32(0.25) * iz)
    r = f32(f32(0.5) * iz)
    lg = f32(np.log2(zl.astype(np.float64)))                      # v_log_f32
    li = np.where(big, _fma32(f32(-HALF_LN2), lg, _fma32(f32(0.125), iz, f32(-HALF_LOG_2PI))), -nli)
    omr = np.where(big, _fma32(e, r, r), omr)
    q = np.where(big, _fma32(f32(0.25), iz, f32(1.0)), q)
    return li, omr, q


def reference(z):
    """float64 values at the float32 arguments."""
    z = np.asarray(z, dtype=np.float64)
    e0, e1 = i0e(z), i1e(z)
    omr = (e0 - e1) / e0
    return np.log(e0), omr, 2.0 * z * omr


def relative_errors(z, values):
    li, omr, q = (np.asarray(v, dtype=np.float64) for v in values)
    rl, ro, rq = reference(z)
    with np.errstate(invalid="ignore", divide="ignore"):
        e_li = np.where(rl != 0.0, np.abs(li - rl) / np.abs(rl), np.abs(li))
        e_omr = np.abs(omr - ro) / ro
        e_q = np.where(rq != 0.0, np.abs(q - rq) / np.abs(rq), np.abs(q))
    return e_li, e_omr, e_q


def test_grid():
    """float32 arguments over [0, 1e5]: zero, a log-spaced sweep, a dense linear
    sweep, and consecutive float32 numbers around the split and at the ends of
    every interval."""
    edges = np.array([_bits(interval(i)[1]) for i in range(N_ENTRY)], np.int64)
    near = (edges[:, None] + np.arange(-4, 4)).reshape(-1)
    near = np.concatenate([near, edges[-1] + np.arange(-64, 64)]).astype(np.uint32).view(f32)
    z = np.concatenate([np.array([0.0], f32), np.geomspace(1e-7, 1e5, 400_000).astype(f32),
                        np.linspace(0.0, 40.0, 400_000).astype(f32), near])
    z = np.unique(z)
    return z[(z >= 0) & (z <= f32(1e5))]


def main(out=None):
    tab = fits()
    z = test_grid()
    e_li, e_omr, e_q = relative_errors(z, evaluate_f32(z, tab))
    print(f"{N_ENTRY} intervals; float32 algorithm over {z.size} arguments in [0, 1e5]: max relative error "
          f"log I0e {e_li.max():.3e} (z={z[e_li.argmax()]:.6g}), 1-R {e_omr.max():.3e} "
          f"(z={z[e_omr.argmax()]:.6g}), q {e_q.max():.3e} (z={z[e_q.argmax()]:.6g}); rms "
          f"{np.sqrt((e_li ** 2).mean()):.2e} {np.sqrt((e_omr ** 2).mean()):.2e} {np.sqrt((e_q ** 2).mean()):.2e}")
    out = out or os.path.join(os.path.dirname(os.path.abspath(__file__)), "bessel_fit.h")
    with open(out, "w") as f:
        f.write("// Generated by gen_bessel_fit.py -- do not edit.\n")
        f.write("// Eq. 9 special functions for 0 <= z < kBesselSplit: per interval of z the expansion\n")
        f.write("// point z0 and the coefficients of -log I0e(z) = c0 + c1 d + ... + c6 d^6, d = z - z0,\n")
        f.write("// whose derivative is 1 - I1(z)/I0(z).  Entry 0 covers [0, 1/8), entry 8 o + i + 1 the\n")
        f.write("// i-th eighth of octave o from 1/8 up.\n")
        f.write(f"// float32 algorithm on the host: log I0e {e_li.max():.2e}, 1-R {e_omr.max():.2e}, "
                f"q {e_q.max():.2e} max relative error over [0, 1e5]\n")
        f.write("#pragma once\n")
        f.write(f"static constexpr int kBesselEntries = {N_ENTRY};\n")
        f.write(f"static constexpr int kBesselShift = {SHIFT};          // entry = (clamped float32 bits - kBesselBitsLo) >> this\n")
        f.write(f"static constexpr int kBesselBitsLo = 0x{BITS_LO:08x};\n")
        f.write(f"static constexpr int kBesselBitsHi = 0x{BITS_HI:08x};\n")
        f.write(f"static constexpr float kBesselFirst = {Z_FIRST!r}f;\n")
        f.write(f"static constexpr float kBesselSplit = {Z_SPLIT!r}f;\n")
        f.write(f"static constexpr float kHalfLog2Pi = {float(f32(HALF_LOG_2PI))!r}f;\n")
        f.write(f"static constexpr float kHalfLn2 = {float(f32(HALF_LN2))!r}f;\n")
        for name, row in zip(["Z0"] + [f"C{k}" for k in range(DEG + 1)], tab):
            vals = [f"{float(f32(v))!r}f" for v in row]
            lines = [", ".join(vals[i:i + 8]) for i in range(0, len(vals), 8)]
            f.write(f"static __device__ const float kBessel{name}[kBesselEntries] = {{" + ",\n    ".join(lines) + "};\n")
    print("wrote", out)


if __name__ == "__main__":
    main()
