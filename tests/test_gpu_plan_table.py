"""The batched writer's table, which the plan makes on the GPU: every element of V is written, at the orders where the
columns a block, the row ranges and the windows change, alone and among other problems."""
import numpy as np
import pytest

from paper_1405_7537_amd import workloads as W

pytestmark = pytest.mark.gpu
EDGES = [1, 2, 31, 32, 33, 127, 128, 255, 256, 257, 511, 512, 513, 1024, 1025, 2047, 2048, 2049, 4096, 4097]


@pytest.mark.parametrize("sizes", [EDGES, EDGES[::-1], [4097], [1] * 3000, [300] * 430, [300] * 432, [2049, 5, 2049]],
                         ids=lambda s: f"{len(s)}x{max(s)}")
def test_every_element_is_written(sizes):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1405_7537_amd.dpr1 as D
    d, z, rho, offs = W.batched(len(sizes), 5, sizes=sizes)
    rho = rho * np.where(np.arange(len(sizes)) % 3 == 1, -1.0, 1.0)
    b = D.Batch(offs)
    b.V.fill_(float("nan"))
    b.solve(*(torch.as_tensor(x, device="cuda") for x in (d, z, rho)))
    b.check()
    assert not bool(b.V.isnan().any())
    # the elements as one problem's writer gives them, within the two solves' rounding of mu and ||x||
    for p in sorted(set([0, len(sizes) // 2, len(sizes) - 1] + (list(range(len(sizes))) if len(sizes) < 30 else []))):
        s = slice(int(offs[p]), int(offs[p + 1]))
        print(f"[plan table] problem {p} n={sizes[p]}", flush=True)
        r = D.eig(d[s], z[s], float(rho[p]))
        assert float(((b.vblock(p) - r.V) / r.V).abs().max()) <= 1e-12
