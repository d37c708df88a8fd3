"""Cells that the row march loads beside its strips, walked on the host for every strip
of many grids: an access past an array's end is one that the range check of the lane's
offset switches off, and every cell that a row uses is the one that was loaded for it."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <algorithm>
#include <cstdio>
#include "flood_rows.h"
using namespace flood;
static long bad = 0, loads = 0;
// the loads for rows r and r + 1 of a strip that ends before row r1
static void load(int ny, int nx, int cw, int ce, int r, int r1, uint32_t es) {
    const uint32_t bytes = (uint32_t)ny * nx * es, so = (uint32_t)r * nx * es;
    for (int lane = 0; lane < 64; ++lane) {
        const uint32_t vo = beside_at(beside_lane(lane) ? beside_cell(lane, nx, cw, ce) * es : kPastEnd, so);
        ++loads;
        if (!beside_lane(lane)) {
            bad += vo < bytes;
            continue;
        }
        const int row = r + (lane == 1 || lane == 62), col = lane < 2 ? cw : ce;
        if (row < r1) bad += vo != ((uint32_t)row * nx + col) * es;       // used
        bad += vo < bytes && vo + es > bytes;
    }
}
int main() {
    for (uint32_t es : {1u, 4u, 8u})
        for (int ny : {1, 2, 3, 5, 8, 63, 64, 65, 130})
            for (int nx : {1, 3, 64, 100})
                for (int rows = 1; rows <= ny; ++rows)
                    for (int r0 = 0; r0 < ny; r0 += rows) {
                        const int r1 = std::min(r0 + rows, ny);
                        load(ny, nx, 0, nx - 1, r0, r1, es);
                        for (int rb = r0; rb < r1; rb += 64)         // pairs of rows, 64 to a block
                            for (int r = rb; r < std::min(rb + 64, r1); r += 2) load(ny, nx, 0, nx - 1, r + 2, r1, es);
                    }
    // the largest arrays: 2^31 bytes, in few and in many rows
    for (int ny : {1, 2, 1 << 14, 1 << 28})
        for (int r = std::max(0, ny - 3); r < ny; ++r) {
            const int nx = (1 << 28) / ny;
            load(ny, nx, nx - 1, 0, r, ny, 8);
            load(ny, nx, nx - 1, 0, r + 2, ny, 8);
        }
    std::printf("%ld loads, %ld bad\n", loads, bad);
    return bad != 0;
}
"""


def test_cells_beside_a_strip_stay_in_their_array(tmp_path):
    src, exe = tmp_path / "rows.cpp", str(tmp_path / "rows")
    src.write_text(SRC)
    b = subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-I",
                        os.path.join(ROOT, "paper_2302_08341_amd", "csrc"), str(src), "-o", exe],
                       capture_output=True, text=True, timeout=120)
    assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
