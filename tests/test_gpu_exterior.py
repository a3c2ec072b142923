"""The exterior eigenvalue when rho ||z||^2 lies far beyond the spread of the poles (penalty-like rank-one terms): mu =
lambda_1 - d_1 against extended precision.  Its equation rho sum z_j^2/(mu + (d_1 - d_j)) = 1 has terms of one sign, so
mu is one rounding from its root (the last sum; 1 eps with the input to it), lambda one more.  Tolerance 2 eps."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
EPS = np.finfo(float).eps
ld = np.longdouble


def exterior(d, z, rho):
    """mu of the exterior eigenvalue, by Newton's steps on the reciprocal of the sum."""
    if rho < 0:
        return -exterior(-d[::-1], z[::-1], -rho)
    delta, z2, r = ld(d[0]) - d.astype(ld), z.astype(ld) ** 2, ld(rho)
    m = r * z2.sum()
    for _ in range(200):
        s, s2 = r * (z2 / (m + delta)).sum(), r * (z2 / (m + delta) ** 2).sum()
        step = s * (s - 1) / s2
        m = m + step
        if abs(step) <= abs(m) * ld(2.0) ** -60:
            break
    return m


@pytest.mark.parametrize("n", [2, 60, 384, 700, 2100])
@pytest.mark.parametrize("vectors", [True, False])
def test_mu_far_beyond_the_poles(n, vectors):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1405_7537_amd.dpr1 as D
    worst = 0.0
    for seed, (spread, rho, zs) in enumerate([(1.0, 1e3, 1.0), (1.0, -1e9, 1.0), (1.0, 1e14, 1.0), (1.0, -1e17, 1.0),
                                              (1.0, 1e20, 1e-3), (1e-20, -1.0, 1.0), (1e-60, 3e2, 1.0),
                                              (1e40, -1e-3, 1e70), (1.0, 1e30, 1e20), (1e-100, 1.0, 1e10),
                                              (1e-6, 1.0, "graded"), (1e-30, -1.0, "graded")]):
        rng = np.random.default_rng(seed)
        d = np.sort(rng.uniform(-1.0, 1.0, n))[::-1] * spread
        z = rng.standard_normal(n) * (1.0 if zs == "graded" else zs)
        if zs == "graded":
            z = z * 10.0 ** rng.uniform(-8, 0, n)
        print(f"[exterior] n={n} spread={spread} rho={rho} z={zs}", flush=True)
        r = D.eig(d, z, rho, vectors=vectors)
        k = 0 if rho > 0 else n - 1
        assert int(r.shift_idx[k]) == k
        m = exterior(d, z, rho)
        e = float(abs(ld(float(r.mu[k])) - m) / abs(m) / EPS)
        lam = ld(d[k]) + m
        el = float(abs(ld(float(r.lam[k])) - lam) / abs(lam) / EPS)
        assert e <= 2.0 and el <= 2.0, (e, el)
        worst = max(worst, e)
    print(f"  worst mu {worst:.2f} eps")
