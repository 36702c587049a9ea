"""Two-interface media at the limits of the image series: the reflection of a round trip
in the finite layer rounds to -1 or +1, where no finite series stands for the density.

For q = -1 the integrals are alternating image sums, which the method of Cohen,
Rodriguez Villegas and Zagier (Convergence acceleration of alternating series, algorithm 1)
sums to a relative 5.8^-n of the integral of the terms' weight from n terms: 40 terms leave
1e-30, so the reference is exact to rounding.  The points lie where the quadrature runs
along the real axis (rho up to the decay length; along the imaginary axis the density has
poles for |q| = 1).  Bound: the quadrature's 1e-12 in interaction units (degree N times
0.87^N R), without a factor 1 / (1 - |q|) because an alternating sum is below its first term.
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

D = [0.0, -1.0]
COMPS = [(lt, ls, a, b) for lt in range(3) for ls in range(3) for a in (1, 2) for b in (1, 2)
         if not (a == 1 and lt == 2) and not (a == 2 and lt == 0)
         and not (b == 1 and ls == 2) and not (b == 2 and ls == 0)]
S, NMAX = 0.25, 8


def _points():
    rng = np.random.default_rng(11)
    rho = np.concatenate([[0.0, 0.3], S * rng.uniform(1.0, 6.0, 14)])
    z = np.concatenate([[0.5, 0.5], S * rng.uniform(1.0, 8.0, 14)])
    return rho, z


def _weight(R):
    w = np.empty((len(R), (NMAX + 1) * (NMAX + 2) // 2))
    for n in range(NMAX + 1):
        w[:, n * (n + 1) // 2:(n + 1) * (n + 2) // 2] = (R * 0.87 ** n)[:, None]
    return w


def _image(rho, Z):
    """S^n (n-m)! P_n^m(Z/R) / R^{n+1} / sqrt((n+m)! (n-m)!) for every n, m <= n."""
    R = np.hypot(rho, Z)
    x, s, t = Z / R, rho / R, S / R
    out = np.zeros((len(rho), (NMAX + 1) * (NMAX + 2) // 2))
    diag = 1.0 / R
    for m in range(NMAX + 1):
        if m > 0:
            diag = diag * t * s * math.sqrt((2 * m - 1) / (2 * m))
        p0, p1 = np.zeros_like(diag), diag
        for n in range(m, NMAX + 1):
            out[:, n * (n + 1) // 2 + m] = p1
            p0, p1 = p1, ((2 * n + 1) * x * t * p1 - math.sqrt(n * n - m * m) * t * t * p0) / math.sqrt((n + 1) ** 2 - m * m)
    return out


def _alternating(rho, Z, step, n=40):
    """sum over j of (-1)^j times the image at Z + j step."""
    d = (3.0 + math.sqrt(8.0)) ** n
    d = (d + 1.0 / d) / 2.0
    b, c, s = -1.0, -d, 0.0
    for k in range(n):
        c = b - c
        s = s + c * _image(rho, Z + k * step)
        b = b * (k + n) * (k - n) / ((k + 0.5) * (k + 1.0))
    return s / d


@pytest.mark.parametrize("eps", [[1e17, 1.0, 1e-17], [1e-17, 1.0, 1e17], [1e20, 1.0, 1e-20]],
                         ids=lambda e: "-".join(f"{v:g}" for v in e))
def test_reflection_of_minus_one(eps):
    from paper_1908_10863_amd import fmmlm as F
    rho, z = _points()
    rt, rb = (eps[1] - eps[0]) / (eps[1] + eps[0]), (eps[1] - eps[2]) / (eps[1] + eps[2])
    assert rt * rb == -1.0
    for (lt, ls, a, b) in COMPS:
        sinf, zi = F.density_asymptotic(D, eps, lt, ls, a, b)
        R = np.hypot(rho, z + zi)
        use = (R >= 2 * S) & (rho <= z + zi)
        got = F.sommerfeld(D, eps, lt, ls, a, b, S, rho, z, NMAX)
        if lt == ls and lt != 1:  # the near interface's reflection, then the waves that cross it
            e0, r = (eps[0], rb) if lt == 0 else (eps[2], rt)
            through = 2.0 * e0 / (e0 + eps[1]) * (2.0 * eps[1] / (e0 + eps[1])) * r
            ref = sinf * _image(rho, z + zi) + through * _alternating(rho, z + zi + 2.0, 2.0)
        else:
            ref = sinf * _alternating(rho, z + zi, 2.0)
        scale = max(1.0, abs(sinf))
        err = np.abs((got - ref) * _weight(R))[use].max()
        assert err <= 1e-12 * scale, (lt, ls, a, b, err)


def test_plan_with_reflection_of_minus_one():
    """Near and far field of a plan.  The same medium with its bottom half space cut by an
    interface between equal permittivities has the same potentials in the other layers (every
    pair on the real axis: the boxes are narrower than a round trip); it has three interfaces
    and is served by the quadrature.  Both plans make the same approximations: 1e-11."""
    import torch
    from paper_1908_10863_amd import fmmlm as F
    rng = np.random.default_rng(4)
    n, eps = 600, [1e17, 1.0, 1e-17]
    x, y = rng.uniform(-0.5, 0.5, (2, n))
    lay = np.repeat([0, 1], n // 2).astype(np.int32)
    z = np.where(lay == 0, rng.uniform(0.05, 0.9, n), rng.uniform(-0.95, -0.05, n))
    q = torch.tensor(rng.uniform(-1, 1, n), device="cuda")
    out = []
    for d, e in ((D, eps), (D + [-2.0], eps + [eps[2]])):
        plan = F.Plan(d, e, x, y, z, lay, p=8, leaf_cap=20, mac_d2=6)
        out.append(plan.eval(q, parts=2).cpu().numpy())
        plan.close()
    assert np.linalg.norm(out[0] - out[1]) <= 1e-11 * np.linalg.norm(out[1])


@pytest.mark.parametrize("eps", [[1e16, 1.0, 1e16], [1.0, 1e16, 1.0], [1.0, 1e17, 1.0]],
                         ids=lambda e: "-".join(f"{v:g}" for v in e))
def test_reflection_of_plus_one(eps):
    """The integral of order 0 diverges in the finite layer: no finite number may come back."""
    from paper_1908_10863_amd import fmmlm as F
    rho, z = _points()
    for (a, b) in ((1, 1), (1, 2), (2, 1), (2, 2)):
        sinf, zi = F.density_asymptotic(D, eps, 1, 1, a, b)
        use = rho <= z + zi
        got = F.sommerfeld(D, eps, 1, 1, a, b, S, rho, z, 0)
        assert not np.isfinite(got[use]).any()


@pytest.mark.parametrize("scale", [2.0 ** 540, 2.0 ** -540])
def test_permittivities_whose_products_leave_the_range(scale):
    """Only ratios of permittivities enter: a common factor, a power of two, changes nothing."""
    from paper_1908_10863_amd import fmmlm as F
    rho, z = _points()
    eps = np.array([2.0, 1.0, 3.0])
    for comp in COMPS:
        np.testing.assert_array_equal(F.sommerfeld(D, eps * scale, *comp, S, rho, z, NMAX),
                                      F.sommerfeld(D, eps, *comp, S, rho, z, NMAX))
