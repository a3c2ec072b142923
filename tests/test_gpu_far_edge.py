"""The accurate pass's part that comes through the far-field expansions, where it is largest: one heavy pole just
beyond the cut (2.5 half-widths of a block's interval, which is 32 gaps wide on either side) and light ones, rho such
that the heavy pole's own eigenvalue falls into a gap of the block.  There the heavy pole gives nearly all of
||x|| and most of the secular sum.  Against extended precision (64-bit mantissa), in units of eps."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
EPS = np.finfo(float).eps
ld = np.longdouble
N, B = 512, 3                                      # eigenvalues 192 .. 255 are the block


@pytest.fixture(scope="module")
def D():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1405_7537_amd.dpr1 as D
    D.lib()
    return D


def solve(D, dist, lane, frac, light, seed):
    """The heavy pole `dist` half-widths below the block's middle, its eigenvalue at `frac` of the gap above pole
    64 B + lane.  Returns errors in eps of (mu, ||x||) of that eigenvalue."""
    rng = np.random.default_rng(seed)
    d = np.linspace(1.0, -1.0, N)
    top, low, k = 64 * B - 1, 64 * B + 63, 64 * B + lane
    c, half = 0.5 * (d[top] + d[low]), 0.5 * (d[top] - d[low])
    h = int(np.argmin(np.abs(d - (c - dist * half))))
    d[h] = c - dist * half
    z = light * rng.uniform(0.5, 1.5, N) * rng.choice([-1.0, 1.0], N)
    z[h] = 1.0
    lam = ld(d[k]) + ld(frac) * (ld(d[k - 1]) - ld(d[k]))
    others = np.arange(N) != h
    s = np.sum(z[others].astype(ld) ** 2 / (d[others].astype(ld) - lam))
    rho = float(-1 / (s + 1 / (ld(d[h]) - lam)))
    r = D.eig(d, z, rho, vectors=False)
    i, mu, xn = int(r.shift_idx[k]), ld(float(r.mu[k])), ld(float(r.xnorm[k]))
    delta, z2, m = d.astype(ld) - ld(d[i]), z.astype(ld) ** 2, mu
    for _ in range(4):
        t = z2 / (delta - m)
        f, fp = 1 + ld(rho) * t.sum(), ld(rho) * (t / (delta - m)).sum()
        m = m - m * f / (f + m * fp)
    nx = np.sqrt((z2 / (delta - m) ** 2).sum())
    assert z2[h] / (delta[h] - m) ** 2 > 0.5 * nx ** 2
    return float(abs(mu - m) / abs(m) / EPS), float(abs(xn - nx) / nx / EPS)


POINTS = [(dist, lane, frac) for dist in (2.502, 2.51, 2.6, 3.0, 4.0)
          for lane, frac in ((0, 0.999), (0, 0.99), (0, 0.9), (0, 0.5), (1, 0.5), (5, 0.4), (20, 0.6), (50, 0.5),
                             (63, 0.1))]


def test_norm_of_a_heavy_pole_beyond_the_cut(D):
    """||x||^2 is the expansions' derivative here.  Its truncation beyond 31 orders is 2^-57 at most; Clenshaw's
    recurrence for the derivative adds up to 4 eps (worst of 15000 points against extended precision), three products
    with |mu| and the half-width 2, the Taylor step and the sum 1: 3.5 eps after the root, which adds 0.5, and the
    division by |mu| and mu's own rounding 1 more: 5."""
    worst = 0.0
    for j, (dist, lane, frac) in enumerate(POINTS):
        print(f"[far edge] norm {dist} lane {lane} at {frac}", flush=True)
        worst = max(worst, solve(D, dist, lane, frac, 1e-6, j)[1])
    print(f"  worst {worst:.2f} eps")
    assert worst <= 5.0


@pytest.mark.parametrize("light", [5e-4, 1e-3])
def test_mu_beside_a_heavy_pole_beyond_the_cut(D, light):
    """The heavy pole is most of the secular sum and of its slope.  The expansions' part is exact to far below eps;
    the light poles' corrected quotients (2 eps) are at most half of the slope: 1 eps; the root's last step and mu =
    s/nu are rounded once each: 1 eps."""
    worst = 0.0
    for j, (dist, lane, frac) in enumerate(POINTS):
        if light * 111 > 0.4 * min(frac, 1 - frac):  # (the gap's own poles would take most of the slope)
            continue
        print(f"[far edge] mu {light} {dist} lane {lane} at {frac}", flush=True)
        worst = max(worst, solve(D, dist, lane, frac, light, j)[0])
    print(f"  worst {worst:.2f} eps")
    assert worst <= 2.0


@pytest.mark.parametrize("n", [500, 1500, 3000])
@pytest.mark.parametrize("near", [0.3, 0.1, 0.01])
def test_exterior_eigenvalue(D, n, near):
    """The exterior eigenvalue's far sums are direct, along the block's threads, and the poles near it lighter than
    the far ones.  mu: the last step and s/nu rounded once each, 1 eps; the terms' errors, 2 eps each at most, average
    over 100 or more: 0.3 eps."""
    worst = 0.0
    for seed in range(12):
        rng = np.random.default_rng(seed)
        d = np.sort(rng.uniform(-1.0, 1.0, n))[::-1].copy()
        z = rng.uniform(0.5, 1.5, n)
        z[:150] *= near
        rho = 10.0 ** rng.uniform(-3, 1)
        r = D.eig(d, z, rho, vectors=False)
        mu = ld(float(r.mu[0]))
        delta, z2, m = d.astype(ld) - ld(d[int(r.shift_idx[0])]), z.astype(ld) ** 2, mu
        for _ in range(4):
            t = z2 / (delta - m)
            f, fp = 1 + ld(rho) * t.sum(), ld(rho) * (t / (delta - m)).sum()
            m = m - m * f / (f + m * fp)
        worst = max(worst, float(abs(mu - m) / abs(m) / EPS))
    print(f"[far edge] exterior n={n} near={near} worst {worst:.2f} eps", flush=True)
    assert worst <= 1.3
