"""Reverse mode where its work is cut over blocks: the pieces of the eigenvalue-only sums."""
import numpy as np
import pytest

from paper_1405_7537_amd import workloads as W

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


@pytest.fixture(scope="module")
def D():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1405_7537_amd.dpr1 as D
    D.lib()
    return D


@pytest.mark.parametrize("nb,n", [(1, 1), (1, 255), (1, 256), (1, 300), (3, 513), (40, 1030), (1, 4099)])
def test_eigenvalue_only_sums_in_pieces(D, nb, n):
    """No V_bar: d_bar, z_bar, rho_bar against the closed form evaluated with NumPy from the forward's
    own V (1 piece, 2, a ragged last piece, several problems), V stored and V rebuilt.  A sum of n terms,
    each with a few roundings (the rebuilt v differs from the stored one by at most 4 eps), is off by at
    most (2 n + 16) eps times the sum of magnitudes."""
    import torch
    dB, zB, rB = W.uniform_batch(nb, n, 50 + n)
    lb = np.random.default_rng(n).standard_normal((nb, n))
    b = D.Batch(np.arange(nb + 1, dtype=np.int64) * n)
    dt, zt, rt, lt = (torch.as_tensor(x, device="cuda") for x in (dB, zB, rB, lb))
    b.solve(dt, zt, rt)
    b.check()
    V = b.V.view(nb, n, n).cpu().numpy()          # [p, k, j]
    xn = b.xnorm.view(nb, n).cpu().numpy()
    tol = (2 * n + 16) * EPS
    for Vin in (b.V, None):
        print(f"[backward] eigenvalue-only nb={nb} n={n} V {'stored' if Vin is not None else 'rebuilt'}", flush=True)
        db, zb, rb = D.backward_batched(dt, zt, rt, b.shift_idx.view(nb, n), b.mu.view(nb, n), b.xnorm.view(nb, n),
                                        Vin, lt, None)
        db, zb, rb = db.cpu().numpy(), zb.cpu().numpy(), rb.cpu().numpy()
        for p in range(nb):
            v2, c = V[p] ** 2, 2.0 * lb[p] / xn[p]
            assert np.max(np.abs(db[p] - lb[p] @ v2) / (np.abs(lb[p]) @ v2)) <= tol
            assert np.max(np.abs(zb[p] + c @ V[p]) / (np.abs(c) @ np.abs(V[p]))) <= tol
            t = lb[p] / (rB[p] * xn[p]) ** 2
            assert abs(rb[p] - t.sum()) <= tol * np.abs(t).sum()


@pytest.mark.parametrize("nb,n", [(1, 1), (1, 129), (3, 257), (9, 128), (17, 40), (2, 1000)])
def test_row_major_v_bar(D, nb, n):
    """V_bar row by row (autograd's layout) gives the bits of the same V_bar column by column, V stored and
    rebuilt, one problem and batches that do not divide over the XCDs."""
    import torch
    dB, zB, rB = W.uniform_batch(nb, n, 70 + n)
    g = torch.Generator(device="cuda").manual_seed(n)
    b = D.Batch(np.arange(nb + 1, dtype=np.int64) * n)
    dt, zt, rt = (torch.as_tensor(x, device="cuda") for x in (dB, zB, rB))
    b.solve(dt, zt, rt)
    b.check()
    lb = torch.randn(nb, n, generator=g, device="cuda", dtype=torch.float64)
    Vb = torch.randn(nb, n, n, generator=g, device="cuda", dtype=torch.float64)      # [p, j, k]
    rep = (b.shift_idx.view(nb, n), b.mu.view(nb, n), b.xnorm.view(nb, n))
    for Vin in (b.V, None):
        print(f"[backward] rows nb={nb} n={n} V {'stored' if Vin is not None else 'rebuilt'}", flush=True)
        cols = D.backward_batched(dt, zt, rt, *rep, Vin, lb, Vb.transpose(1, 2).contiguous())
        rows = D._backward_batched(dt, zt, rt, *rep, Vin, lb, Vb, n, 1)
        for x, y in zip(cols, rows):
            assert torch.equal(x, y)
    # one problem, V_bar a slice of wider rows, against the column-major call
    r = [t[0].contiguous() for t in rep]
    V = b.V[: n * n].view(n, n).t()
    wide = torch.randn(n, n + 3, generator=g, device="cuda", dtype=torch.float64)[:, :n]
    one = D.backward(dt[0], zt[0], float(rB[0]), *r, V, lb[0], wide)
    ref = D.backward(dt[0], zt[0], float(rB[0]), *r, V, lb[0], wide.t().contiguous().t())
    for x, y in zip(one, ref):
        assert torch.equal(x, y)
