"""The tuner's memory of measured geometries, built on the host without a device: a
geometry serves the kind of catchments and the step kernel that it was measured with."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2302_08341_amd", "csrc")

SRC = r"""
#include <cstdio>
#include "flood_tune.h"
using namespace flood;
static int bad = 0;
#define EXPECT(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); ++bad; } } while (0)
int main() {
    TuneKey plain{};
    plain.real_bytes = 4;
    plain.n_catch = 2;
    for (int i = 0; i < 2; ++i) plain.ny[i] = 53 + i, plain.nx[i] = 72, plain.members[i] = 4;
    TuneKey land = plain, inflow = plain, other = plain;
    land.kind[0] = 1;
    inflow.kind[1] = 2;
    other.kind[1] = 1;
    TuneChoice c, got;
    c.variant = 3;
    c.march_rows = 1;
    c.march_narrow = 1;
    EXPECT(!tune_lookup(plain, 1, 0, got));
    tune_store(plain, c);
    EXPECT(tune_lookup(plain, 1, 0, got) && got.march_rows == 1 && got.march_narrow == 1);
    EXPECT(tune_lookup(plain, 1, 3, got));
    EXPECT(!tune_lookup(plain, 1, 1, got) && !tune_lookup(plain, 1, 2, got));
    EXPECT(!tune_lookup(land, 1, 0, got) && !tune_lookup(inflow, 1, 0, got));
    c.march_rows = 16;
    c.march_narrow = 0;
    tune_store(land, c);
    EXPECT(tune_lookup(land, 1, 0, got) && got.march_rows == 16);
    EXPECT(!tune_lookup(other, 1, 0, got));
    EXPECT(tune_lookup(plain, 1, 0, got) && got.march_rows == 1);
    std::printf("%d bad\n", bad);
    return bad;
}
"""
# a file written before: plain keys, without and with the last field
OLD = """b4_mi1_53x72x4_54x72x4 1 4 4 3 1 1 1 1,1 1
b4_mi1_53x72x4l_54x72x4 1 4 4 3 8 1 4 8,8
"""
SRC_FILE = r"""
#include <cstdio>
#include "flood_tune.h"
using namespace flood;
int main() {
    TuneKey k{};
    k.real_bytes = 4;
    k.n_catch = 2;
    for (int i = 0; i < 2; ++i) k.ny[i] = 53 + i, k.nx[i] = 72, k.members[i] = 4;
    TuneChoice g;
    if (!tune_lookup(k, 1, 0, g) || g.march_rows != 1 || g.march_narrow != 1) return 1;
    if (tune_lookup(k, 1, 2, g)) return 2;
    k.kind[0] = 1;
    if (!tune_lookup(k, 1, 0, g) || g.march_rows != 8 || g.march_narrow != -1 || g.march_order != 4) return 3;
    k.kind[0] = 2;
    return tune_lookup(k, 1, 0, g) ? 4 : 0;
}
"""


def _run(tmp_path, src, **env):
    cpp, exe = tmp_path / "tune.cpp", str(tmp_path / "tune")
    cpp.write_text(src)
    b = subprocess.run(["g++", "-std=c++17", "-Wall", "-O1", "-I", CSRC, str(cpp), os.path.join(CSRC, "flood_tune.cpp"),
                        "-o", exe], capture_output=True, text=True, timeout=120)
    assert b.returncode == 0, b.stderr[-4000:]
    clean = {k: v for k, v in os.environ.items() if not k.startswith("FLOOD_")}
    return subprocess.run([exe], capture_output=True, text=True, timeout=60, env=dict(clean, **env))


def test_a_geometry_serves_what_it_was_measured_with(tmp_path):
    r = _run(tmp_path, SRC)
    assert r.returncode == 0, r.stdout


def test_the_same_from_a_file(tmp_path):
    f = tmp_path / "cache.txt"
    f.write_text(OLD)
    r = _run(tmp_path, SRC_FILE, FLOOD_TUNE_CACHE=str(f))
    assert r.returncode == 0, r.returncode
    # and what one process stores, another finds
    f.unlink()
    assert _run(tmp_path, SRC, FLOOD_TUNE_CACHE=str(f)).returncode == 0
    assert f.read_text().count("\n") == 2


def test_strip_heights(tmp_path):
    r = _run(tmp_path, r"""
#include "flood_tune.h"
using flood::strip_heights;
using V = std::vector<int>;
int main() {
    if (strip_heights(0, false) != V{2, 4, 8, 16, 32, 64} || strip_heights(0, true) != V{4, 8, 16, 32, 64}) return 1;
    // with land cover from the rows of the drained volume's sums on, each catchment's too
    for (bool refine : {false, true})
        if (strip_heights(4, refine) != V{4, 8, 16, 32, 64} || strip_heights(8, refine) != V{8, 16, 32, 64}) return 2;
    return 0;
}
""")
    assert r.returncode == 0, r.returncode


def test_where_strips_of_one_cell_a_lane_compete(tmp_path):
    r = _run(tmp_path, r"""
#include "flood_tune.h"
using namespace flood;
static bool competes(int rb, int ny, int nx, int n) {
    TuneKey k{};
    k.real_bytes = rb;
    k.n_catch = 1;
    k.ny[0] = ny, k.nx[0] = nx, k.members[0] = n;
    return narrow_competes(k);
}
int main() {
    // few wavefronts
    if (!competes(4, 97, 83, 5) || !competes(4, 128, 256, 128) || !competes(8, 256, 128, 64)) return 1;
    // many, on grids that leave lanes idle: rows shorter than a strip, or just past one
    if (!competes(4, 1000, 48, 40) || !competes(4, 1000, 128, 40) || !competes(4, 300, 301, 96)) return 2;
    if (!competes(8, 1000, 64, 40) || !competes(4, 4096, 1, 1024)) return 3;
    // many, with the lanes in use
    if (competes(4, 1000, 256, 40) || competes(4, 2000, 2000, 96) || competes(4, 1000, 224, 40)) return 4;
    if (competes(8, 1000, 128, 40) || competes(4, 701, 503, 96)) return 5;
    return 0;
}
""")
    assert r.returncode == 0, r.returncode
