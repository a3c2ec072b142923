"""CPU tests of the sizes of the far-field expansions (paper_1405_7537_amd/csrc/far_sizes.h): launches and
workspaces at every order that the interface accepts."""
import ctypes as C
import os
import subprocess

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
    for f in (L.shim_far_blocks, L.shim_far_records, L.shim_far_room, L.shim_far_block_threads):
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
