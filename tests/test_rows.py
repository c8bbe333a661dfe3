"""Row arithmetic of the planning kernels (csrc/rows.hpp), compiled for the host: whatever the offsets hold, positions stay inside
the tables.  The header is the one the kernels include; the program walks the groups as the planning workgroup does."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "rows.hpp"
// first positions of S * E groups in expert-major order, by passes of 16 wavefronts of 64 lanes; saturated sums, or plain 32-bit ones
template <bool SATURATED> std::vector<int> positions(const std::vector<int32_t>& off, int S, int E, int M) {
    auto add = [&](int a, int b) { return SATURATED ? add_rows(a, b, M) : (int)((unsigned)a + (unsigned)b); };
    std::vector<int> pos(S * E + 1);
    int base = 0;
    for (int i0 = 0; i0 < S * E; i0 += 1024) {
        int wave_tot[16], excl[1024];
        for (int w = 0; w < 16; ++w) {
            int incl[64], next[64];
            for (int l = 0; l < 64; ++l) {
                const int i = i0 + 64 * w + l;
                int lo;
                incl[l] = i < S * E ? group_rows(off.data(), (i % S) * E + i / S, M, lo) : 0;
            }
            for (int step = 1; step < 64; step <<= 1) {
                for (int l = 0; l < 64; ++l) next[l] = l >= step ? add(incl[l], incl[l - step]) : incl[l];
                for (int l = 0; l < 64; ++l) incl[l] = next[l];
            }
            for (int l = 0; l < 64; ++l) excl[64 * w + l] = l ? incl[l - 1] : 0;
            wave_tot[w] = incl[63];
        }
        int before = 0;
        for (int w = 0; w < 16; ++w) {
            for (int l = 0; l < 64; ++l)
                if (i0 + 64 * w + l < S * E) pos[i0 + 64 * w + l] = add(base, add(before, excl[64 * w + l]));
            before = add(before, wave_tot[w]);
        }
        base = add(base, before);
    }
    pos[S * E] = base;
    return pos;
}
int main(int argc, char** argv) {
    const int S = atoi(argv[2]), E = atoi(argv[3]), M = atoi(argv[4]);
    std::vector<int32_t> off(S * E + 1);
    FILE* f = fopen(argv[1], "rb");
    if (!f || fread(off.data(), 4, off.size(), f) != off.size()) return 2;
    const auto a = positions<true>(off, S, E, M), b = positions<false>(off, S, E, M);
    fwrite(a.data(), 4, a.size(), stdout);
    fwrite(b.data(), 4, b.size(), stdout);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    (d / "rows.cpp").write_text(PROGRAM)
    subprocess.run([shutil.which("g++") or "c++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2605_26845_amd", "csrc"), str(d / "rows.cpp"),
                    "-o", str(d / "rows")], check=True)
    return d


def positions(program, offsets, S, E, M):
    (program / "offsets").write_bytes(offsets.astype(np.int32).tobytes())
    out = np.frombuffer(subprocess.run([str(program / "rows"), str(program / "offsets"), str(S), str(E), str(M)], check=True, capture_output=True).stdout,
                        dtype=np.int32)
    return out[: S * E + 1], out[S * E + 1:]


def exact(offsets, S, E, M):
    o = offsets.astype(np.int64)
    lo = np.clip(o[:-1], 0, M)
    rows = np.maximum(np.minimum(o[1:], M), lo) - lo
    return np.minimum(np.concatenate([[0], np.cumsum(rows.reshape(S, E).T.ravel())]), M)


@pytest.mark.parametrize("S,E,M", [(1, 1, 7), (3, 2, 100), (300, 4, 5000), (2, 2050, 6000), (16384, 4, 72408)])
def test_positions_of_ordinary_offsets(program, S, E, M):
    offsets = np.sort(np.random.default_rng(S + E).integers(0, M + 1, S * E + 1))
    offsets[0] = 0
    saturated, plain = positions(program, offsets, S, E, M)
    assert np.array_equal(saturated, exact(offsets, S, E, M)) and np.array_equal(saturated, plain)


@pytest.mark.parametrize("S,E,M", [(16384, 4, 72408), (1, 65536, 72408), (65536, 1, 65537), (512, 2, 8 << 20), (40, 3, (1 << 31) - 1)])
def test_positions_of_malformed_offsets_stay_inside(program, S, E, M):
    """Groups that each claim every row: plain 32-bit sums wrap below zero here, where the row list would be written outside."""
    offsets = np.tile([0, M], S * E)[: S * E + 1]
    saturated, plain = positions(program, offsets, S, E, M)
    assert plain.min() < 0
    assert saturated.min() >= 0 and saturated.max() <= M and (np.diff(saturated) >= 0).all()
    assert np.array_equal(saturated, exact(offsets, S, E, M))
    for other in (-offsets, offsets[::-1].copy(), np.random.default_rng(S).integers(-(1 << 31), 1 << 31, S * E + 1)):
        saturated, _ = positions(program, other, S, E, M)
        assert np.array_equal(saturated, exact(other, S, E, M))
