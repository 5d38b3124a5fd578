"""The order in which a launch's workgroups take its (head, item) units: map_unit of csrc/device_common.h with the
host's table, compiled for the CPU as it stands in the sources."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_04421_amd", "csrc")
CUS = 256
KINDS = ["fwd", "causal fwd", "dq", "dkdv"]

PROGRAM = """
#include "kernels.h"
#include "schedule.h"
#define __device__
#define __forceinline__ inline
static inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
namespace hmar {
%s
}
extern "C" unsigned units(int n_items, int n_heads, int batch_groups, int reverse, int* head, int* item) {
    const unsigned n = hmar::launch_groups(n_items, n_heads);
    if (!head) return n;
    const hmar::UnitMap m = hmar::unit_map_for(n_items, n_heads, batch_groups);
    for (unsigned wg = 0; wg < n; ++wg) hmar::map_unit((int)wg, m, head + wg, item + wg, reverse != 0);
    return n;
}
const hmar::Order orders[] = {hmar::kOrderFwd, hmar::kOrderFwdCausal, hmar::kOrderDq, hmar::kOrderDkDv};
extern "C" int batch_groups(int n_items, int n_heads, int cus, int kind) {
    return hmar::launch_map(cus, n_items, n_heads, orders[kind]).batch_grouped / 8;
}
extern "C" unsigned launch_units(int n_items, int n_heads, int cus, int reverse, int kind, int* head, int* item) {
    const unsigned n = hmar::launch_groups(n_items, n_heads);
    if (!head) return n;
    const hmar::UnitMap m = hmar::launch_map(cus, n_items, n_heads, orders[kind]);
    for (unsigned wg = 0; wg < n; ++wg) hmar::map_unit((int)wg, m, head + wg, item + wg, reverse != 0);
    return n | (m.turned ? 1u << 31 : 0);
}
extern "C" int one_launch(int n_q, int n_k, int max_q, int max_k, int total, int n_heads, int cus) {
    hmar::DeviceSchedule s{};
    s.n_items[0] = n_q; s.n_items[1] = n_k; s.max_tiles[0] = max_q; s.max_tiles[1] = max_k;
    s.total_tiles[0] = total / 2; s.total_tiles[1] = total - total / 2; s.num_cus = cus;
    return hmar::one_backward_launch(s, n_heads);
}
extern "C" int ahead(int max_tiles, int long_items, int n_heads, int cus) { return hmar::keys_ahead(max_tiles, long_items, n_heads, cus); }
extern "C" int whole_rows(int kind, long long units, int max_tiles, int cus) {
    return kind == 0 ? hmar::whole_rows_fwd(units, cus) : kind == 1 ? hmar::whole_rows_dq(units, max_tiles, cus)
                                                                    : hmar::whole_rows_dkdv(units, max_tiles, cus);
}
extern "C" int last_long(const int* tiles, int n) {
    std::vector<hmar::TileItem> items;
    for (int i = 0; i < n; ++i) items.push_back({0, 1, 64 * i, 64 * (i + tiles[i]) - 63 * (i & 1)});
    return hmar::items_to_last_long(items);
}
extern "C" int quotient(int n, int d) { return hmar::divide(n, d, hmar::inverse_of(d)); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("unit_map")
    text = open(os.path.join(CSRC, "device_common.h")).read()
    begin = text.index("__device__ __forceinline__ int divide(")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text("#pragma once\n#include <cstddef>\ntypedef int hipError_t; typedef void* hipStream_t;\n")
    (d / "map.cpp").write_text(PROGRAM % text[begin:text.index("__device__ __forceinline__ void map_workgroup(")])
    cmd = [shutil.which("g++") or "g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", str(d), "-I", CSRC, str(d / "map.cpp"), os.path.join(CSRC, "schedule.cpp"),
           "-o", str(d / "map.so")]
    subprocess.run(cmd, check=True)
    return ctypes.CDLL(str(d / "map.so"))


def _units(lib, n_items, n_heads, batch_groups, reverse=False):
    n = lib.units(n_items, n_heads, 1, 0, None, None)
    head, item = np.zeros(n, np.int32), np.zeros(n, np.int32)
    p = lambda a: a.ctypes.data_as(ctypes.POINTER(ctypes.c_int))
    lib.units(n_items, n_heads, batch_groups, int(reverse), p(head), p(item))
    return head, item


def _launch_units(lib, n_items, n_heads, cus, kind, reverse=False):
    """(heads, items, whether the second units are dealt backwards) of the workgroups of a launch."""
    n = n_items * n_heads
    head, item = np.zeros(n, np.int32), np.zeros(n, np.int32)
    p = lambda a: a.ctypes.data_as(ctypes.POINTER(ctypes.c_int))
    lib.launch_units.restype = ctypes.c_uint
    back = lib.launch_units(n_items, n_heads, cus, int(reverse), KINDS.index(kind), p(head), p(item)) >> 31
    return head, item, back


def _batch(n_items, n_heads, cus, kind):
    """Groups of eight heads in the batch that ends a launch: eight units for every compute unit of an XCD, half of them for
    lists of up to seven items and, where the batch would be the whole launch, up to fifteen in the backward; the whole
    launch where less than a unit per compute unit would be left ahead of it.  The forward under the block-causal mask:
    never half."""
    groups, full = n_heads // 8, max(1, cus // 8 * 8 // n_items)
    half = kind != "causal fwd" and (n_items < 8 or (n_items < 16 and full >= groups and kind != "fwd"))
    batch = min(groups, max(1, full // 2) if half else full)
    return groups if (groups - batch) * n_items < cus // 8 else batch


@pytest.mark.parametrize("batch_groups", [1, 2, 7, 40, 1000])         # 1: a single step of items that are alike
@pytest.mark.parametrize("reverse", [False, True])
@pytest.mark.parametrize("n_items", [1, 2, 3, 5, 7, 8, 20, 70, 255, 256, 257, 1000])
def test_every_unit_has_one_workgroup(lib, n_items, reverse, batch_groups):
    for n_heads in list(range(1, 42)) + [48, 63, 100, 104, 107] + ([768, 1023, 1536] if n_items < 100 else [300]):
        head, item = _units(lib, n_items, n_heads, batch_groups, reverse)
        assert len(head) == n_items * n_heads
        assert head.min() >= 0 and head.max() < n_heads and item.min() >= 0 and item.max() < n_items
        assert np.bincount(head.astype(np.int64) * n_items + item, minlength=n_items * n_heads).max() == 1
        # a head of a whole group keeps to the XCD of its number
        xcd, grouped = np.arange(len(head)) % 8, head < n_heads // 8 * 8
        assert (head[grouped] % 8 == xcd[grouped]).all()


def _assert_order(head, item, n_items, n_heads, batch, reverse):
    # whole groups head by head, the last `batch` of them item by item
    groups = n_heads // 8
    slot, xcd = np.arange(len(head)) // 8, np.arange(len(head)) % 8
    first = (groups - batch) * n_items
    group = np.where(slot < first, slot // n_items, groups - batch + (slot - first) % batch)
    assert (item == np.where(slot < first, slot % n_items, (slot - first) // batch)).all()
    assert (head == (groups - 1 - group if reverse else group) * 8 + xcd).all()


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n_items,n_heads", [(7, 768), (20, 192), (7, 256), (8, 256), (12, 200), (12, 480), (1, 4096), (70, 48), (300, 16)])
def test_whole_groups_are_walked_head_by_head_and_the_last_batch_item_by_item(lib, n_items, n_heads, kind):
    for reverse in (False, True):
        head, item, back = _launch_units(lib, n_items, n_heads, CUS, kind, reverse)
        assert not back
        _assert_order(head, item, n_items, n_heads, _batch(n_items, n_heads, CUS, kind), reverse)


@pytest.mark.parametrize("n_items,n_heads", [(2, 1536), (5, 600), (12, 48)])
def test_a_step_of_items_that_are_alike_is_walked_head_by_head(lib, n_items, n_heads):
    _assert_order(*_units(lib, n_items, n_heads, 1), n_items, n_heads, 1, False)


@pytest.mark.parametrize("cus", [256, 304, 64])
@pytest.mark.parametrize("kind", KINDS)
def test_every_unit_of_a_launch_has_one_workgroup(lib, kind, cus):
    turned, turn = 0, 2 if kind == "dkdv" else 6
    for n_items in [1, 2, 3, 7, 8, 9, 15, 16, 20, 31, 70, 300]:
        for n_heads in list(range(1, 42)) + [63, 64, 72, 100, 104, 160, 256, 288, 768, 1023]:
            for reverse in (0, 1):
                n = n_items * n_heads
                head, item, back = _launch_units(lib, n_items, n_heads, cus, kind, reverse)
                assert np.array_equal(np.sort(head.astype(np.int64) * n_items + item), np.arange(n))
                xcd, grouped = np.arange(n) % 8, head < n_heads // 8 * 8
                assert (head[grouped] % 8 == xcd[grouped]).all()
                assert not back or cus < n <= turn * cus
                if back:        # first unit of a compute unit heavy to light, second light to heavy
                    for x in range(8):
                        mine, c = item[x::8], cus // 8
                        assert (np.diff(mine[:c]) >= 0).all() and (np.diff(mine[c:2 * c]) <= 0).all()
                turned += back
    assert turned > 0


@pytest.mark.parametrize("kind", KINDS)
def test_the_batch_that_ends_a_launch(lib, kind):
    for cus in (256, 304):
        for n_items in (1, 3, 7, 8, 11, 15, 16, 20, 300):
            for n_heads in list(range(1, 60)) + list(range(60, 700, 13)) + [768, 1536]:
                got = lib.batch_groups(n_items, n_heads, cus, KINDS.index(kind))
                assert got == _batch(n_items, n_heads, cus, kind), (n_items, n_heads, cus)


@pytest.mark.parametrize("tiles,tenths", [(1, 20), (7, 20), (25, 20), (32, 20), (33, 18), (64, 18)])
def test_a_backward_is_one_launch_up_to_its_line(lib, tiles, tenths):
    # work for two of the longest items on every compute unit; on streams of 33 tiles and more 9/5 of them (up to
    # 2 took 3 % longer in one launch than in two, at worst 14 %)
    for cus in (256, 304):
        line = tenths * tiles * cus // 10
        assert lib.one_launch(3, 3, tiles, tiles, line, 1, cus) and not lib.one_launch(3, 3, tiles, tiles, line + 1, 1, cus)
        assert lib.one_launch(3, 3, tiles, 1, line // 8, 8, cus) and not lib.one_launch(3, 3, 1, tiles, line // 8 + 1, 8, cus)
        assert not lib.one_launch(3, 4, tiles, tiles, line, 1, cus)          # lists of one length only
        assert not lib.one_launch(3, 3, tiles, 65, 1, 1, cus) and lib.one_launch(3, 3, 65, tiles, 1, 1, cus)


def test_own_rows_are_asked_for_whole_up_to_one_line(lib):
    # the fuller the launch and the longer its streams, the less whole rows pay: one line in each direction, no gap
    lib.whole_rows.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    for cus in (256, 304):
        for kind, rounds in ((0, 3), (1, 3), (2, 2)):
            for tiles in (1, 7, 8, 15, 16, 64):
                whole = [lib.whole_rows(kind, units, tiles, cus) for units in (1, rounds * cus, rounds * cus + 1, 5 * cus, 7 * cus, 1 << 33)]
                assert whole == [1, 1] + 4 * [int(kind > 0 and tiles < 16)], (kind, tiles)


def test_key_operands_are_asked_for_ahead_where_no_two_long_chains_share_a_compute_unit(lib):
    for cus in (256, 304):
        for tiles in (1, 15, 16, 64):
            short = int(tiles < 16)
            assert [lib.ahead(tiles, 2, h, cus) for h in (1, cus // 2, cus // 2 + 1, cus, cus + 1, 9 * cus)] == [1, 1, 0, 0, short, short]
        assert not lib.ahead(15, 1 << 14, 1 << 18, cus) == lib.ahead(16, 1 << 14, 1 << 18, cus)          # beyond 32 bits
    for tiles, n in (([7, 7, 4, 7, 5, 3, 3], 5), ([3], 1), ([5, 5, 5], 3), ([10, 7, 6, 6], 2), ([10, 6, 6, 1], 1), ([6, 1, 1, 10], 4)):
        assert lib.last_long((ctypes.c_int * len(tiles))(*tiles), len(tiles)) == n, tiles


def test_quotients_by_the_inverse(lib):
    rng = np.random.default_rng(1)
    for d in [1, 2, 3, 7, 8, 255, 256, 641, 16384] + rng.integers(1, 1 << 20, 50).tolist():
        for n in [0, 1, d - 1, d, d + 1, 5 * d - 1, 5 * d, (1 << 31) - 1, (1 << 31) - 1 - (1 << 31) % d] + rng.integers(0, 1 << 31, 50).tolist():
            assert lib.quotient(int(n), int(d)) == n // d, (n, d)
