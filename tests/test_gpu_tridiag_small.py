"""Every order that the divide and conquer does not split (a block's round robin has its rows rounded up to even),
against eigenvalues bisected in extended precision, with the tolerances of one block: 2 eps ||T|| for the
eigenvalues, 8 for orthogonality and residual where no eigenvalues are closer than 2^-20 ||T||."""
import numpy as np
import pytest

from test_gpu_tridiag_leaf import EPS, bisected, ld, matrix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["random", "one_two_one"])
def test_every_small_order(kind):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1405_7537_amd.dpr1 as D
    for n in range(1, 33):
        print(f"[small] {kind} n={n}", flush=True)
        a, b = matrix(kind, n)
        r = D.tridiag_eig(a, b)
        lam, Q = r.lam.cpu().numpy().astype(ld), r.Q.cpu().numpy().astype(ld)
        ref = bisected(a, b)
        nt = np.max(np.abs(ref))
        T = (np.diag(a) + np.diag(b, 1) + np.diag(b, -1)).astype(ld)
        assert np.max(np.abs(lam - ref)) <= 2 * EPS * nt
        if n > 1 and np.min(ref[:-1] - ref[1:]) < nt * 2.0 ** -19:
            continue
        assert np.max(np.abs(Q.T @ Q - np.eye(n))) <= 8 * EPS
        assert np.max(np.abs(T @ Q - Q * lam)) <= 8 * EPS * nt
