"""How the score kernel's batches are cut into stretches (csrc/tri_items.h, no GPU needed): every tile in one stretch, a head-instance's
pieces in entries of their own that the workspace has room for, and where the lines of the rule lie."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256
WRAPPER = """
#include "tri_items.h"
using namespace tri;
extern "C" {
int rounds(int G, long long instances, int n, int n_cu) { return stretch_rounds(G, instances, n, n_cu); }
int least(long long instances, int n, long long stretches) { return stretch_least(instances, n, stretches); }
int entries(int n, int least) { return stretch_entries(n, least); }
unsigned count(unsigned total, unsigned least, unsigned most) { return stretches_of(total, least, most).count; }
unsigned wanted(unsigned total, unsigned longest, unsigned entries, unsigned most, unsigned n_cu, unsigned waves)
{
    return stretches_wanted(total, longest, entries, most, n_cu, waves);
}
int own(int id, int grid, int stretches) { return own_stretch(id, grid, stretches); }
unsigned begin(unsigned total, unsigned least, unsigned most, unsigned i) { return stretch_begin(stretches_of(total, least, most), i); }
unsigned of(unsigned total, unsigned least, unsigned most, unsigned tile) { return stretch_of(stretches_of(total, least, most), tile); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("stretches")
    src, so = str(tmp / "s.cpp"), str(tmp / "s.so")
    with open(src, "w") as f:
        f.write(WRAPPER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_2604_04921_amd", "csrc"),
                    src, "-o", so], check=True)
    so = ctypes.CDLL(so)
    so.rounds.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    so.least.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_longlong]
    for f in (so.count, so.begin, so.of):
        f.restype = ctypes.c_uint
    return so


def test_every_tile_once_and_room_for_the_moments(lib):
    rng = random.Random(11)
    taken = 0
    for _ in range(400):
        n, seqs, lh = int(2 ** rng.uniform(0, 17)), rng.randint(1, 12), rng.randint(1, 300)
        r = lib.rounds(4, lh * seqs, n, CUS)
        if r == 0:
            continue
        taken += 1
        most = r * CUS
        least = lib.least(lh * seqs, n, most)
        entries = lib.entries(n, least)
        assert entries <= -(-n // 256) + 1   # an entry per 256 keys and one more: what workspaces are sized for
        lens = [rng.choice([0, 1, n, rng.randint(0, n), rng.randint(0, n)]) for _ in range(seqs)]
        tiles = [-(-x // 64) for x in lens]
        total = sum(tiles) * lh
        count = lib.count(total, least, most)
        assert count <= most and (count > 0) == (total > 0)
        starts = [lib.begin(total, least, most, i) for i in range(count + 1)]
        assert starts[0] == 0 and starts[-1] == total if total else True
        sizes = [b - a for a, b in zip(starts, starts[1:])]
        assert max(sizes) - min(sizes) <= 1 if sizes else True
        at = 0
        for _ in range(min(lh, 3)):
            for t in tiles:
                if t:
                    first = lib.of(total, least, most, at)
                    last = lib.of(total, least, most, at + t - 1)
                    assert starts[first] <= at < starts[first + 1] and starts[last] <= at + t - 1 < starts[last + 1]
                    assert last - first + 1 <= entries, (n, least, t)
                at += t
    assert taken > 100


@pytest.mark.parametrize("group,instances,n,stretches", [
    (4, 121, 2176, True), (4, 120, 2176, False),             # more than sixteen tiles per CU
    (4, 2047, 2176, True), (4, 2048, 2176, False),           # short sequences: not in large batches
    (4, 2047, 32768, True), (4, 2048, 32768, False),         # 32 items per CU and more
    (4, 2304, 8192, True), (4, 8192, 8192, False),
    (8, 511, 32768, True), (8, 512, 32768, False)])          # more than four query heads: not in large batches
def test_where_the_lines_lie(lib, group, instances, n, stretches):
    assert (lib.rounds(group, instances, n, CUS) > 0) == stretches


def test_the_number_that_the_lengths_ask_for(lib):
    """Lengths up to the reserved one, and far below it: every stretch has a tile, and a head-instance's lie in as many as it has entries for."""
    rng = random.Random(12)
    taken = 0
    for _ in range(600):
        n, seqs, lh = int(2 ** rng.uniform(0, 17)), rng.randint(1, 12), rng.randint(1, 300)
        r = lib.rounds(4, lh * seqs, n, CUS)
        if r == 0:
            continue
        taken += 1
        most = r * CUS
        entries = lib.entries(n, lib.least(lh * seqs, n, most))
        top = rng.choice([n, n, rng.randint(0, n), int(n ** rng.random())])
        tiles = [-(-x // 64) for x in (rng.choice([0, 1, top, rng.randint(0, top), rng.randint(0, top)]) for _ in range(seqs))]
        total = sum(tiles) * lh
        count = lib.wanted(total, max(tiles), entries, most, CUS, rng.choice([8, 12]))
        assert count <= min(most, total) and (count > 0) == (total > 0)
        assert count % CUS == 0 or count < CUS
        at = 0
        for _ in range(min(lh, 3)):
            for t in tiles:
                if t:
                    assert lib.of(total, 1, count, at + t - 1) - lib.of(total, 1, count, at) + 1 <= entries, (n, count, t)
                at += t
    assert taken > 100


@pytest.mark.parametrize("instances,tiles,n", [
    (8, 34, 131072), (288, 34, 131072), (72, 34, 131072), (512, 16, 32768), (512, 1, 1665), (136, 3, 2547), (288, 128, 32768), (1152, 64, 32768)])
def test_lengths_far_below_the_reserved_one(lib, instances, tiles, n):
    """Every CU has its share of the tiles that there are, also where max_seq_len says little about them."""
    most, total = lib.rounds(4, instances, n, CUS) * CUS, instances * tiles
    assert most > 0
    count = lib.wanted(total, tiles, lib.entries(n, lib.least(instances, n, most)), most, CUS, 12)
    assert -(-count // CUS) * -(-total // count) <= 1.15 * -(-total // CUS) + 1, count   # tiles of the CU that has the most


@pytest.mark.parametrize("instances,tiles,waves,slots", [(1056, 39, 8, 2), (1056, 40, 8, 2), (1008, 41, 8, 2), (2016, 34, 8, 2), (1584, 40, 12, 2), (1152, 64, 12, 2),
                                                         (2016, 20, 12, 4), (2016, 13, 12, 4)])
def test_every_workgroup_has_its_share(lib, instances, tiles, waves, slots):
    """The stretches that workgroups end up with where some of them are one item and others, of more pieces than an item holds, two: each item in the time
    of its tiles (and seven), the number of a later stretch asked for at the beginning of an item, where the next one is its stretch's last."""
    total, n = instances * tiles, tiles * 64
    count = lib.wanted(total, tiles, lib.entries(n, lib.least(instances, n, lib.rounds(8, instances, n, CUS) * CUS)), lib.rounds(8, instances, n, CUS) * CUS,
                       CUS, waves)
    assert count % CUS == 0

    def items(i):   # tiles of the items of stretch i
        at, end, sizes = lib.begin(total, 1, count, i), lib.begin(total, 1, count, i + 1), []
        while at < end:
            cut = min(end, (at // tiles + 1) * tiles)
            sizes.append(cut - at)
            at = cut
        return [sum(sizes[j:j + slots]) for j in range(0, len(sizes), slots)]

    counter, taken = 2 * CUS, [[w] for w in range(CUS)]
    listed = [[(t, w) for t in items(w)] for w in range(CUS)]   # the items that a workgroup knows of
    last = list(range(CUS))
    clock = [(0, w) for w in range(CUS)]
    while clock:
        now, w = min(clock)
        clock.remove((now, w))
        while last[w] < count and len(listed[w]) < 3:   # the item at hand, the next one, the one after it
            if lib.own(last[w], CUS, count):
                nxt = last[w] + CUS
            else:
                nxt, counter = counter, counter + 1
            last[w] = nxt
            if nxt < count:
                taken[w].append(nxt)
                listed[w] += [(t, nxt) for t in items(nxt)]
        if listed[w]:
            clock.append((now + listed[w].pop(0)[0] + 7, w))
    assert sorted(i for t in taken for i in t) == list(range(count))
    assert all(len(t) == count // CUS for t in taken), sorted(set(len(t) for t in taken))
