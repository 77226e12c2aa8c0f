"""The launches of the affine chains stay within HIP's limit of fewer than 2^32
work-items (csrc/launch_limits.h), on the CPU."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1304_6514_amd", "csrc")

SOURCE = r"""
#include "launch_limits.h"
using namespace nv::lin;
extern "C" {
int products(int M, long long N) { return products_fit(M, N); }
int states(int M, long long N, long long Q, long long from) { return states_fit(M, N, Q, from); }
long long groups(long long Q, int paired) { return many_groups(Q, paired); }
int paired(int M, long long Q, long long blocks, long long from) {
    return many_paired(M, Q, blocks, from);
}
long long rows(long long blocks, int product) { return many_rows(blocks, product); }
int by_blocks(long long N, long long Q, int cus) { return states_by_blocks(N, Q, cus); }
}
"""
PAIR_FROM = 2 * 256 * 32


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("limits")
    (d / "limits.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    str(d / "limits.cpp"), "-o", str(d / "limits.so")], check=True)
    lib = ctypes.CDLL(str(d / "limits.so"))
    ll = ctypes.c_longlong
    lib.products.argtypes = [ctypes.c_int, ll]
    lib.states.argtypes = [ctypes.c_int, ll, ll, ll]
    lib.groups.argtypes, lib.groups.restype = [ll, ctypes.c_int], ll
    lib.paired.argtypes = [ctypes.c_int, ll, ll, ll]
    lib.rows.argtypes, lib.rows.restype = [ll, ctypes.c_int], ll
    lib.by_blocks.argtypes = [ll, ll, ctypes.c_int]
    return lib


def items(lib, M, N, Q, product):
    """Work-items of the launch over every block of 8 of N maps."""
    blocks = (N + 7) // 8
    paired = not product and lib.paired(M, Q, blocks, PAIR_FROM)
    return lib.groups(M + 1 if product else Q, paired) * lib.rows(blocks, product) * 512


@pytest.mark.parametrize("M", [1, 2, 15, 16, 99, 104, 105, 127])
def test_a_launch_by_blocks_is_taken_exactly_where_it_fits(lib, M):
    for N in (64, 71, 1024, 1025, 60000, 1 << 20, 33_554_432, 67_108_800, 67_108_863):
        assert lib.products(M, N) == (items(lib, M, N, 0, True) < 2 ** 32), (M, N)
        for Q in (1, 16, 17, 300, 16384, 131072, 1_048_576, 1_100_000, 2_097_152, 2_200_000,
                  100_000_000, 1 << 31):
            assert lib.states(M, N, Q, PAIR_FROM) == (items(lib, M, N, Q, False) < 2 ** 32), \
                (M, N, Q)
    # 2,200,000 chains of 1024 slices: one launch over the blocks does not hold them
    assert not lib.states(M, 1024, 2_200_000, PAIR_FROM)


def test_many_chains_with_states_run_slice_by_slice(lib):
    for N, most in ((64, 12), (95, 12), (96, 24), (127, 24), (128, 32), (1 << 20, 32)):
        assert lib.by_blocks(N, most * 256, 256) and not lib.by_blocks(N, most * 256 + 1, 256)


def test_every_block_has_its_groups(lib):
    """The numbers of a launch, block by block or in turns over eight dies, cover every
    (block, group) once (the kernel's own arithmetic)."""
    for blocks in (1, 2, 8, 9, 13):
        for product in (0, 1):
            rows, groups = lib.rows(blocks, product), 3
            spread = 8 if product and blocks > 1 else 1
            seen = set()
            for wg in range(rows * groups):
                turn = wg // spread
                block, group = turn // groups * spread + wg % spread, turn % groups
                if block < blocks:
                    assert (block, group) not in seen
                    seen.add((block, group))
            assert len(seen) == blocks * groups
