"""The eigenvector writer of one problem at the edges of its tiles (512 positions by 8 columns), for
columns that start on 128-byte lines and for every offset from one (leading dimension, buffer).

Both forms evaluate the same expression on the same values, so V is compared bit for bit with that of
an aligned buffer, whose columns are checked against the quotients in numpy: the writer's quotient is
corrected to 1 ulp, one more rounding each for the product with zeta and for 1/||x||, and the
difference d_j - sigma - mu is the same in both; 4 eps relative.
"""
import ctypes

import numpy as np
import pytest

from paper_1405_7537_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1405_7537_amd.dpr1 as D
    D.lib()
    return D


def solve(D, d, z, rho, ldv, shift, vwrite=0):
    """V [n, n] (columns), sigma index, mu, ||x|| from a buffer whose first column starts `shift`
    doubles behind a 256-byte boundary; what lies between and around the columns must stay."""
    import torch
    n = len(d)
    dev = dict(dtype=torch.float64, device="cuda")
    td, tz = torch.tensor(d, **dev), torch.tensor(z, **dev)
    lam, mu, xn = (torch.empty(n, **dev) for _ in range(3))
    idx = torch.empty(n, dtype=torch.int32, device="cuda")
    info = torch.empty(1, dtype=torch.int32, device="cuda")
    buf = torch.full((32 + ldv * n + 64,), -7.25, **dev)
    lib, opts = D.lib(), D.Opts()
    lib.dpr1_default_opts(ctypes.byref(opts))
    opts.vwrite = vwrite
    wb = int(lib.dpr1_workspace_size(n))
    work = torch.empty(wb, dtype=torch.uint8, device="cuda")
    rc = lib.dpr1_eig(D._ptr(td), D._ptr(tz), float(rho), n, D._ptr(lam), buf.data_ptr() + 8 * (32 + shift), ldv,
                      D._ptr(idx), D._ptr(mu), D._ptr(xn), D._ptr(info), None, ctypes.byref(opts), D._ptr(work), wb,
                      D._stream())
    assert rc == 0 and int(info.item()) == 0
    b = buf.cpu().numpy()
    cols = b[32 + shift:32 + shift + ldv * n].reshape(n, ldv)
    assert np.all(b[:32 + shift] == -7.25) and np.all(b[32 + shift + ldv * n:] == -7.25)
    assert np.all(cols[:, n:] == -7.25)
    return cols[:, :n].T.copy(), idx.cpu().numpy(), mu.cpu().numpy(), xn.cpu().numpy()


@pytest.mark.parametrize("rho", [1.0, -0.5])
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 510, 511, 512, 513, 527, 528, 1024, 1025, 1040])
def test_tile_edges(D, n, rho):
    d, z, _ = W.uniform(n, n)
    print(f"[tiles] n={n} rho={rho}", flush=True)
    V, idx, mu, xn = solve(D, d, z, rho, (n + 15) // 16 * 16, 0)
    want = z[:, None] / (((d[:, None] - d[idx][None, :]) - mu[None, :]) * xn[None, :])
    assert np.max(np.abs(V - want) / np.abs(want)) <= 4 * np.finfo(float).eps
    for ldv, shift in [(n, 0), (n + 1, 0), (n + 2, 3), (n + 15, 15), ((n + 15) // 16 * 16, 1),
                       ((n + 15) // 16 * 16 + 16, 8)]:
        assert np.array_equal(solve(D, d, z, rho, ldv, shift)[0], V), (ldv, shift)


@pytest.mark.parametrize("rho", [1.0, -0.5])
def test_written_in_chunks(D, rho):
    """The chunked writer (a range of columns per launch) at an order off every edge."""
    d, z, _ = W.uniform(8197, 4)
    ref = solve(D, d, z, rho, 8208, 0)[0]
    for ldv, shift, chunks in [(8208, 0, 3), (8197, 0, 3), (8198, 5, 8)]:
        assert np.array_equal(solve(D, d, z, rho, ldv, shift, chunks)[0], ref), (ldv, shift, chunks)


@pytest.mark.parametrize("mean", ["small", "large"])
def test_batch_blocks(D, mean):
    """A batch's blocks: columns per block and windows at the orders where either changes, on both
    sides of the rule for the blocks that finish flagged eigenpairs."""
    import torch
    sizes = [1, 2, 31, 32, 33, 126, 127, 128, 129, 255, 256, 257, 511, 512, 513]
    if mean == "large":
        sizes += [1023, 1025, 2047, 2048, 2049, 2300]
    print(f"[tiles] batch {mean}", flush=True)
    offs = np.concatenate([[0], np.cumsum(sizes)])
    data = [W.uniform(n, 50 + n) for n in sizes]
    d, z = (np.concatenate([x[i] for x in data]) for i in range(2))
    rho = np.array([0.75 if i % 2 else -1.5 for i in range(len(sizes))])
    b = D.Batch(offs, vectors=True)
    r = b.solve(*(torch.tensor(x, dtype=torch.float64, device="cuda") for x in (d, z, rho)))
    torch.cuda.synchronize()
    idx, mu, xn = (x.cpu().numpy() for x in (r.shift_idx, r.mu, r.xnorm))
    for p, n in enumerate(sizes):
        s = slice(offs[p], offs[p + 1])
        V = b.vblock(p).cpu().numpy()
        dp, zp = d[s], z[s]
        want = zp[:, None] / (((dp[:, None] - dp[idx[s]][None, :]) - mu[s][None, :]) * xn[s][None, :])
        assert np.max(np.abs(V - want) / np.abs(want)) <= 4 * np.finfo(float).eps, n
