// Offsets of the cells that the row march reads beside a strip.  Plain functions of
// integers, for the kernels and for the host.
#pragma once

#include <cstdint>

namespace flood {

// lane offset of a buffer access that is switched off: past the end of every array
// (2^31 bytes at most), also with a row's offset added
constexpr uint32_t kPastEnd = 0xc0000000u;

// Lanes 0 and 63 take the cells west (column cw) and east (ce) of a strip in row r,
// lanes 1 and 62 those in row r + 1: the cell's index, from the start of row r.
constexpr bool beside_lane(int lane) { return lane < 2 || lane > 61; }
constexpr uint32_t beside_cell(int lane, uint32_t nx, uint32_t cw, uint32_t ce) {
    return lane < 2 ? (uint32_t)lane * nx + cw : (uint32_t)(63 - lane) * nx + ce;
}
// The offset of row r (row) added to that of a lane, held at the largest value.  These
// loads run up to three rows ahead of the row in work and so past the grid's last
// row: their whole offset is the lane's, which the range check of a buffer covers
// (it does not have to cover a scalar one).
constexpr uint32_t beside_at(uint32_t lane_offset, uint32_t row) {
    const uint32_t at = lane_offset + row;
    return at < lane_offset ? 0xffffffffu : at;
}

}  // namespace flood
