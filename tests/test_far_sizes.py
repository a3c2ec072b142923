"""CPU tests of the sizes of the far-field expansions (paper_1405_7537_amd/csrc/far_sizes.h): launches and
workspaces at every order that the interface accepts."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("shim") / "libfar_sizes_shim.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared",
                           os.path.join(HERE, "host", "far_sizes_shim.cpp"), "-o", out])
    L = C.CDLL(out)
    for f in (L.shim_far_blocks, L.shim_far_records, L.shim_far_room):
        f.argtypes = [C.c_int64]
    L.shim_far_batch_own.argtypes, L.shim_far_batch_wide.argtypes = [C.c_int64] * 3, [C.c_int64] * 2
    for f in (L.shim_far_blocks, L.shim_far_records, L.shim_far_room, L.shim_far_block_threads, L.shim_far_min,
              L.shim_far_batch_own, L.shim_far_batch_wide):
        f.restype = C.c_int64
    return L


@pytest.mark.parametrize("n", [384, 2048, 32768, 10 ** 6, 2 ** 23 - 64, 2 ** 23, 2 ** 26 + 1, (2 ** 31 - 1) // 2])
def test_launch_fits(shim, n):
    """A launch has fewer than 2^32 threads."""
    blocks = shim.shim_far_blocks(n)
    assert 0 < blocks and blocks * shim.shim_far_block_threads() < 2 ** 32


def test_workspace_is_linear_and_grows(shim):
    """At most 240 bytes a row at every order from 4096 on, and never less for more rows: the wide records fit in their room."""
    from paper_1405_7537_amd import dpr1 as D
    orders = sorted({o + k for e in range(9, 27) for o in (2 ** e, 3 * 2 ** (e - 1)) for k in (-512, -65, -1, 0, 1, 513)})
    orders += list(range(30000, 140000, 509))
    last = (0, 0)
    for n in sorted(set(orders)):
        size = D.workspace_bytes(n)
        assert n < 4096 or size <= 240 * n, n
        assert size >= last[1], (n, last)
        assert shim.shim_far_records(n) <= shim.shim_far_room(n), n
        last = (n, size)


BATCHES = [[4096], [2048], [2049], [383] * 9, [384], [384] * 500, [385] * 40, [16] * 1000 + [40000], [2047, 2048, 1],
           [2049] * 64, [32768, 32769], [65536], [14337] * 3, [511, 2559, 33281]]
BATCHES += [np.random.default_rng(s).integers(1, 10 ** (1 + s % 4), 30).tolist() + [3000] * (s % 2) for s in range(16)]


@pytest.mark.parametrize("sizes", BATCHES, ids=lambda s: f"{len(s)}x{max(s)}")
def test_batch_room_holds_the_records(shim, sizes):
    N, nmax, items = sum(sizes), max(sizes), sum((n + 63) // 64 for n in sizes)
    own = sum((n + 63) // 64 for n in sizes if n >= shim.shim_far_min())
    assert own <= shim.shim_far_batch_own(N, nmax, N // 64 + len(sizes)) and items <= N // 64 + len(sizes)
    assert sum(shim.shim_far_records(n) for n in sizes) <= shim.shim_far_batch_wide(N, nmax)


@pytest.mark.parametrize("sizes", [[4096], [2048, 16, 16], [384, 100], [100, 7], [2200, 500]],
                         ids=lambda s: f"{len(s)}x{max(s)}")
@pytest.mark.parametrize("short", [1, 1000])
def test_batched_solve_refuses_a_short_workspace(sizes, short):
    """dpr1_eig_batched is handed the plan and the workspace's size: less than the size query's answer is -15, before
    anything is launched (the pointers are never followed)."""
    from paper_1405_7537_amd import dpr1 as D
    L = D.lib()
    offs = (C.c_int64 * (len(sizes) + 1))(0, *np.cumsum(sizes).tolist())
    need = L.dpr1_batched_workspace_size(len(sizes), offs)
    o = D.Opts()
    L.dpr1_default_opts(C.byref(o))
    plan = D.Plan(len(sizes), sum(sizes), sum((n + 63) // 64 for n in sizes), max(sizes), 0, 1, 1, o)
    p = C.c_void_p(0x1000)
    # (ngroups = 0: 2048 entries of the table count at least; 550 x 2 + 32 is the most of these batches)
    rc = L.dpr1_eig_batched(C.byref(plan), p, p, p, p, p, None, None, None, None, None, p, None, p, need - short, None)
    assert rc == -15
