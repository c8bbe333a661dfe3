"""Parts of the weight gradients' contractions (csrc/parts.hpp), compiled for the host: the table has room for every call that the entry point takes.
The header is the one the kernel includes; one thread, or seven with a barrier, do here what the workgroup does there."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS, MAX_UNITS = 256, 1024
PROGRAM = r"""
#include <barrier>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <thread>
#include <vector>
#include "parts.hpp"
struct Entry { int x, y, z, w; };
int main(int argc, char** argv) {
    const int E = atoi(argv[2]), tiles = atoi(argv[3]), cus = atoi(argv[4]), cap = atoi(argv[5]);
    int n = 1;
    while (n < E) n *= 2;
    std::vector<int> bases(E + 1);
    FILE* f = fopen(argv[1], "rb");
    if (!f || fread(bases.data(), 4, bases.size(), f) != bases.size()) return 2;
    const size_t room = 1 + dw_entries(E);
    std::vector<Entry> entries(room + 64 * (size_t)E, Entry{-7, -7, -7, -7});          // (what lies behind the table is looked at too)
    std::vector<Entry> alone = entries;
    for (int threads : {1, 7}) {
        std::vector<int> rows(n), order(n), parts(E), sums(threads);
        std::barrier<> all(threads);
        std::vector<std::thread> group;
        std::fill(entries.begin(), entries.end(), Entry{-7, -7, -7, -7});
        for (int t = 0; t < threads; ++t)
            group.emplace_back([&, t] {
                dw_split(bases.data(), E, tiles, cus, cap, entries.data(), rows.data(), order.data(), parts.data(), sums.data(), t, threads, [&] { all.arrive_and_wait(); });
            });
        for (std::thread& t : group) t.join();
        if (threads == 1) alone = entries;
        if (memcmp(alone.data(), entries.data(), 16 * entries.size())) return 3;
    }
    fwrite(&room, 8, 1, stdout);
    fwrite(entries.data(), 16, entries.size(), stdout);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("parts")
    (d / "parts.cpp").write_text(PROGRAM)
    subprocess.run([shutil.which("g++") or "c++", "-O1", "-std=c++20", "-pthread", "-I", os.path.join(ROOT, "paper_2605_26845_amd", "csrc"), str(d / "parts.cpp"),
                    "-o", str(d / "parts")], check=True)
    return d


def tiles_of(d, f):
    return f // 128 * (d // 256) + d // 256 * -(-f // 256)


def split(program, rows, tiles, cap=MAX_UNITS):
    """-> per part (position, rows, expert, part, parts of the expert, first place), after every check that the table allows."""
    bases = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    (program / "bases").write_bytes(bases.tobytes())
    out = subprocess.run([str(program / "parts"), str(program / "bases"), str(len(rows)), str(tiles), str(CUS), str(cap)], check=True, capture_output=True).stdout
    room, table = int(np.frombuffer(out, np.int64, 1)[0]), np.frombuffer(out, np.int32, offset=8).reshape(-1, 4)
    n = int(table[0, 0])
    assert 1 + 2 * n <= room and (table[1 + 2 * n:] == -7).all()          # nothing lies behind the table, nothing behind the entries
    e = np.concatenate([table[1:1 + 2 * n:2], table[2:2 + 2 * n:2, :2]], axis=1)
    # every expert once, with most rows first; its parts follow each other and cover its rows
    at, taken = 0, []
    for expert in sorted(range(len(rows)), key=lambda j: (-rows[j], j)):
        parts, place = int(e[at, 4]), int(e[at, 5])
        own = e[at:at + parts]
        assert (own[:, 2] == expert).all() and (own[:, 3] == np.arange(parts)).all() and (own[:, 4] == parts).all() and (own[:, 5] == place).all()
        assert own[0, 0] == bases[expert] and (own[1:, 0] == own[:-1, 0] + own[:-1, 1]).all() and own[:, 1].sum() == rows[expert] and (own[:, 1] >= 0).all()
        if parts > 1:
            taken.append((place, place + parts * tiles))
        at += parts
    assert at == n
    taken.sort()
    assert all(0 <= lo and hi <= cap for lo, hi in taken) and all(a[1] <= b[0] for a, b in zip(taken, taken[1:]))
    return e


def steps(first, equal, growth):
    """Rows per expert, slowly rising: `equal` experts of `first` rows, then growth[k] from one to the next while the rows are within e^(k / 2) ..
    e^((k + 1) / 2) times the first ones; as many experts as the entry point takes."""
    rows = [first] * equal
    while True:
        k = min(len(growth) - 1, int(2 * np.log(rows[-1] / first)))
        rows.append(int(np.ceil(rows[-1] * growth[k])))
        if sum(rows) + 256 * len(rows) >= 1 << 22:
            return rows[:-1]


# (one place per part asked for and none refused, these make 1025 to 1080 parts more than experts)
MANY = [steps(4276, 42, [1.01244, 1.01278, 1.01292, 1.01294, 1.0124, 1.00904]), steps(6370, 52, [1.01269, 1.01252, 1.013, 1.01284, 1.01167, 1.01076])]


@pytest.mark.parametrize("rows", MANY + [MANY[0][::-1], steps(1800, 78, [1.013]), [25000] * 85])
def test_table_of_many_experts(program, rows):
    """Every expert is long beside the work behind it and asks to be split: more parts than the table and the places for their sums hold."""
    e = split(program, rows, tiles_of(256, 256))
    assert (e[:, 4] > 1).any() and len(e) <= len(rows) + MAX_UNITS


@pytest.mark.parametrize("cap", [0, 1, 5, 6, 7, 100, 1024])
def test_no_room_for_sums(program, cap):
    """Too few places: the experts that find none stay whole, one entry each."""
    e = split(program, [40000, 30000, 30000, 20000, 5000, 0, 1], 3, cap)
    assert cap >= 6 or (e[:, 4] == 1).all()


@pytest.mark.parametrize("seed", range(40))
def test_random_experts(program, seed):
    rng = np.random.default_rng(seed)
    E = int(rng.choice([1, 2, 4, 8, 60, 300, 1000]))
    rows = rng.multinomial(int(rng.integers(1, 3_900_000)), rng.dirichlet(np.full(E, rng.choice([0.3, 1.0, 10.0]))))
    split(program, rows, tiles_of(256 * int(rng.integers(1, 9)), 128 * int(rng.integers(2, 12))), int(rng.choice([0, 40, 1024])))


def test_parts_of_one_expert(program):
    """One expert of 136 tiles on 256 compute units: whole below twice 768 rows; the round of units that ends first above."""
    assert [len(split(program, [n], tiles_of(2048, 1408))) for n in (1, 1535)] == [1, 1]
    assert len(split(program, [36833], tiles_of(2048, 1408))) > 1
    assert len(split(program, [100000], tiles_of(256, 256))) == 32
