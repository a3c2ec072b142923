"""The reduction of the front end on the GPU (sort, groups, compaction, order of the columns) at the
edges of its runs of 512 rows and its passes of 16 runs, against the same reduction in numpy
followed by the direct solve.

Tolerances: eigenvalues to 1e-13 relative (the reduced z differs by the order in which a group's
squares are added, n eps at most, as much for the eigenvalue's distance to its pole; deflated poles
exactly); V^T V - I to (20 + n) eps (entries to 10 eps relative, a sum of n products); A V - V Lambda
to (20 + n) eps (max|d| + |rho| |z|^2), entry by entry, for the same reasons.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
EPS = np.finfo(float).eps


def inputs(kind, n, seed):
    rng = np.random.default_rng(seed)
    d, z = rng.standard_normal(n), rng.standard_normal(n)
    if kind == "pairs":  # pairs and zeros everywhere
        k = rng.permutation(n)[: n - n % 2].reshape(2, -1)
        half = k.shape[1] // 3
        d[k[0, :half]] = d[k[1, :half]]
        z[rng.random(n) < 0.2] = 0.0
    elif kind == "few":  # groups of many runs' length, one of them without z
        v = rng.standard_normal(7)
        j = rng.integers(0, 7, n)
        d = v[j]
        z[j == 3] = 0.0
    elif kind == "equal":
        d[:] = -0.75
    elif kind == "zeros":  # +0 and -0 are one pole; nothing else enters the reduced problem
        d[::2], z[1::2] = np.where(rng.random(d[::2].size) < 0.5, 0.0, -0.0), 0.0
    elif kind == "deflated":
        z = z * 2.0 ** -520
    elif kind == "sorted":
        d = np.sort(d)[::-1].copy()
    elif kind == "ascending":
        d = np.sort(d)
    return d, z


def reduced(d, z):
    """Decreasing poles and z of the reduced problem, and the deflated or reflected eigenvalues."""
    z = np.where(np.abs(z) < 2.0 ** -511, 0.0, np.abs(z))
    v, inv = np.unique(-(d + 0.0), return_inverse=True)
    s = np.bincount(inv, weights=z * z)
    cnt = np.bincount(inv)
    keep = s > 0
    rest = np.repeat(-v, cnt - keep)
    return -v[keep], np.sqrt(s[keep]), rest


KINDS = ["pairs", "few", "equal", "zeros", "deflated", "sorted", "ascending"]


@pytest.mark.parametrize("hermitian", [False, True])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [1, 2, 64, 65, 511, 512, 513, 1025, 8192, 8193])
def test_edges(n, kind, hermitian):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1405_7537_amd.dpr1 as D
    rho = -1.25 if n % 2 else 0.5
    d, z = inputs(kind, n, n)
    zz = z * np.exp(1j * np.random.default_rng(n + 1).uniform(0, 6.28, n)) if hermitian else z
    print(f"[front] {kind} n={n} hermitian={hermitian}", flush=True)
    r = (D.eig_hermitian if hermitian else D.eig_general)(d, zz, rho)
    lam = r.lam.cpu().numpy()
    rd, rz, rest = reduced(d, np.abs(zz))
    solved = D.eig(rd, rz, rho, vectors=False).lam.cpu().numpy() if rd.size else np.empty(0)
    want = np.sort(np.concatenate([rest, solved]))[::-1]
    el = np.max(np.abs(lam - want) / np.where(want == 0, 1.0, np.abs(want)))
    V, dd, zd = r.V, torch.tensor(d, device="cuda"), torch.tensor(zz, device="cuda")
    eye = torch.eye(n, dtype=V.dtype, device="cuda")
    eo = (V.conj().t().contiguous() @ V - eye).abs().max().item()
    AV = dd[:, None] * V + rho * zd[:, None] * (zd.conj()[None, :] @ V)
    er = (AV - V * r.lam[None, :]).abs().max().item() / (np.max(np.abs(d)) + abs(rho) * np.sum(np.abs(zz) ** 2) + 1e-300)
    print(f"  reduced to {rd.size}: lambda {el:.1e} V^T V {eo:.1e} residual {er:.1e}", flush=True)
    assert el <= 1e-13 and eo <= (20 + n) * EPS and er <= (20 + n) * EPS


def test_three_passes_values():
    """More than 16 x 16 runs: a third pass; eigenvalues only."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1405_7537_amd.dpr1 as D
    d, z = inputs("pairs", 131585, 5)
    lam = D.eig_general(d, z, 1.0, vectors=False).lam.cpu().numpy()
    rd, rz, rest = reduced(d, z)
    want = np.sort(np.concatenate([rest, D.eig(rd, rz, 1.0, vectors=False).lam.cpu().numpy()]))[::-1]
    assert np.max(np.abs(lam - want) / np.abs(want)) <= 1e-13


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("at", [0, 511, 512, 8192])
def test_not_finite_anywhere(at, value):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1405_7537_amd.dpr1 as D
    for which in range(2):
        x = inputs("pairs", 8193, 9)
        x[which][at] = value
        with pytest.raises(ValueError, match="non-finite"):
            D.eig_general(*x, 1.0)
        with pytest.raises(ValueError, match="non-finite"):
            D.eig_hermitian(x[0], x[1] + 0j, 1.0)
