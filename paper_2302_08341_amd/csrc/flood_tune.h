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
bool tune_enabled();
// The choice remembered for a problem, for a handle that names step kernel
// step_kernel (0: leaves it open): a geometry is that of the kernel it was measured
// with, and of the extensions in the key (the row march's strips may be one cell
// wide and one row tall for plain catchments, which no other form takes).
bool tune_lookup(const TuneKey& k, int mi, int step_kernel, TuneChoice& out);
void tune_store(const TuneKey& k, const TuneChoice& c);

}  // namespace flood
