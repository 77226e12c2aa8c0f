"""The staging rings of the composition chains (csrc/chain_ring.h), on the CPU:
every slot of a ring is filled by one wave only, so that a late load of one wave
never lands in what another has staged."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1304_6514_amd", "csrc")

SOURCE = r"""
#include "chain_ring.h"
using namespace nv::dev;
extern "C" {
void layout(int n, int comps, int elem, int *out) {
    const PfLayout l(n, comps, elem);
    const int v[] = {l.rows, l.width, l.slots, l.helpers, l.row_bytes, l.slot_bytes, l.ahead,
                     l.lds_bytes()};
    for (int i = 0; i < 8; ++i) out[i] = v[i];
}
int staged(int count, int cus) { return batch_staged(count, cus); }
void constants(int *out) {
    const int v[] = {kPfPair, kPfHelpers, kPfMaxSlots, kPfRingBytes, kPf2Slots, kPf2Ahead, kPfWin, kPfBesideBuild};
    for (int i = 0; i < 8; ++i) out[i] = v[i];
}
}
"""
TABLES = [(comps, elem) for comps in (1, 2) for elem in (4, 8)]
# every row up to well past the line between rows and windows, and longer ones
SIZES = [*range(2, 4200), 8191, 65536, 1 << 20]


class Ring:
    def __init__(self, lib, n, comps, elem):
        out = (ctypes.c_int * 8)()
        lib.layout(n, comps, elem, out)
        (self.rows, self.width, self.slots, self.helpers, self.row_bytes, self.slot_bytes,
         self.ahead, self.lds) = out


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("ring")
    (d / "ring.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    str(d / "ring.cpp"), "-o", str(d / "ring.so")], check=True)
    return ctypes.CDLL(str(d / "ring.so"))


@pytest.fixture(scope="module")
def const(lib):
    out = (ctypes.c_int * 8)()
    lib.constants(out)
    return dict(zip(("pair", "helpers", "max_slots", "ring_bytes", "slots2", "ahead2", "window", "beside"), out))


@pytest.mark.parametrize("comps,elem", TABLES)
def test_every_slot_has_one_owner(lib, const, comps, elem):
    for n in SIZES:
        r = Ring(lib, n, comps, elem)
        assert 1 <= r.helpers <= const["helpers"] and r.slots <= const["max_slots"]
        owner = {}
        for s in range(6 * r.slots):                  # slices, from the range's first
            wave = (s // const["pair"]) % r.helpers
            assert owner.setdefault(s % r.slots, wave) == wave, (n, s)
        # a slot is filled when the slice before it in the slot is finished
        assert 0 < r.ahead < r.slots
        assert r.slots * r.slot_bytes <= const["ring_bytes"]


def test_every_slot_of_the_bilinear_ring_has_one_owner(const):
    owner = {}
    for s in range(6 * const["slots2"]):
        wave = s % const["helpers"]
        assert owner.setdefault(s % const["slots2"], wave) == wave
    assert const["ahead2"] < const["slots2"]


@pytest.mark.parametrize("comps,elem", TABLES)
def test_a_window_holds_the_narrowest_one_and_its_slack(lib, const, comps, elem):
    """A helper stages a window of at least kPfWin nodes, or none: a slot that is
    narrower would never serve a slice."""
    seen = 0
    for n in SIZES:
        r = Ring(lib, n, comps, elem)
        assert r.row_bytes >= r.width * elem + 15 and r.row_bytes % 16 == 0   # any alignment
        assert r.slot_bytes == comps * r.row_bytes
        if not r.rows:
            seen += 1
            assert const["window"] <= r.width < n
            assert r.slots > r.ahead
    assert seen


@pytest.mark.parametrize("comps,elem", TABLES)
def test_the_ring_takes_what_the_table_needs(lib, const, comps, elem):
    """Never more LDS than lies above the granules of eight build workgroups (a chain
    that overlaps a build starts beside five of them), about 64 KB for windows of up to
    8 bytes per node and for rows of up to 4 KB."""
    for n in SIZES:
        r = Ring(lib, n, comps, elem)
        assert r.slots * r.slot_bytes + 64 < r.lds <= const["beside"]
        if (not r.rows and comps * elem <= 8) or n * comps * elem <= 4000:
            assert r.lds <= 67 * 1024
        assert r.slots <= 16 or r.rows


def test_a_batch_is_staged_up_to_two_problems_per_cu(lib):
    assert lib.staged(1, 256) and lib.staged(512, 256) and not lib.staged(513, 256)
