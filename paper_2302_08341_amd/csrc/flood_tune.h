// Kernel-geometry tuner of libflood: the key of a tuning problem, the chosen
// geometry, the defaults used before (or instead of) measuring, and a small
// text cache of measured choices.
#pragma once

#include <vector>

namespace flood {

struct TuneKey {
    int real_bytes;
    int n_catch;
    int ny[8], nx[8], members[8];
    int kind[8];         // of a catchment: bit 0 land cover, bit 1 inflow links
};

struct TuneChoice {
    int mi = 1;          // members interleaved in the fastest index
    int tile_rows = 4;   // cell rows per 256-lane tile
    int cpb = 16;        // member chunks per workgroup
    int variant = 1;     // 1 tiled kernel, 2 row-marching kernel, 3 vectorised row march
    int march_rows = 32; // rows per strip of the row-marching kernel
    int march_seg = 2;   // members marched together by one wavefront
    int march_order = 1; // wavefront order of the row-march kernels (0 to 4)
    int march_narrow = -1; // vectorised row march: 1 strips of one cell a lane, 0 of whole vectors, -1 by rule
    int march_rows_c[8] = {0, 0, 0, 0, 0, 0, 0, 0};   // per catchment, 0: march_rows
};

TuneChoice tune_default(const TuneKey& k);
// Strip heights that the vectorised row march is tried at, and again for each of
// several catchments (refine).  drain_rows: with land cover, the rows that the drained
// volume is summed over (0: none); its strips are whole numbers of them, so that the
// sum is the same for every height.
std::vector<int> strip_heights(int drain_rows, bool refine);
// Whether strips of one cell a lane compete with those of whole vectors (16 bytes of
// cells a lane) for plain catchments: while the chip holds all the wavefronts of the
// latter, two rows tall, and where these leave more than a fifth of their lanes idle
// beside the grid.  A pass over 60 s in FP32, vectors against one cell a lane, ms: 40
// members of 1000 x 48 3.32 and 1.66, 1000 x 97 3.80 and 2.56, 1000 x 128 3.58 and 2.62, 1000 x
// 160 3.79 and 3.69, 1000 x 192 (three quarters of the lanes in use) 3.71 and 3.57; 300 x 301
// x 96 5.47 and 4.21.  A step of 1000 x 224 x 40 (seven eighths) 40 and 44 us: from there on
// one cell a lane pays on few wavefronts only.
bool narrow_competes(const TuneKey& k);
bool tune_enabled();
// The choice remembered for a problem, for a handle that names step kernel
// step_kernel (0: leaves it open): a geometry is that of the kernel it was measured
// with, and of the extensions in the key (the row march's strips may be one cell
// wide and one row tall for plain catchments, which no other form takes).
bool tune_lookup(const TuneKey& k, int mi, int step_kernel, TuneChoice& out);
void tune_store(const TuneKey& k, const TuneChoice& c);

}  // namespace flood
