// Address arithmetic of the conv patch kernels that the host checks too:
// plain constexpr functions, without HIP.
#pragma once

namespace xtc {

// 16-byte units that hold `bytes` bytes from `mis` bytes into the first one.
constexpr int units_of(int mis, int bytes) { return (mis + bytes + 15) >> 4; }

// A run of input rows (one image's, in one channel plane) is copied in 16-byte
// units.  Its slot holds the units of the worst 2-byte position; a channel's
// own position may need one fewer, and that one would start where the run
// ends, for the last plane of the tensor past its memory.
constexpr int slot_units(int bytes) { return bytes > 0 ? units_of(14, bytes) : 0; }

// Entry of the unit table: position of the unit in its run and the length of
// the run, both in bytes and below 2^15; negative past the last run.
constexpr int unit_entry(int u, int bytes) { return bytes << 16 | u * 16; }

// Byte offset of that unit where the run starts at byte `start`, `oob` where
// the run does not reach it.
constexpr int unit_offset(int entry, int start, int oob) {
    return entry >= 0 && (entry & 0xffff) < (start & 15) + (entry >> 16) ? (start & ~15) + (entry & 0xffff) : oob;
}

// Lane and scalar offset (bytes) of the store of one output, `row` bytes past
// the lane's first one at `first`; `whole`: every output channel of the tile
// exists.  A store that does not exist goes to an offset past the buffer, which
// drops it: the sum must stay below 2^32, and `row` itself (27 channel planes)
// may be past 2^31 where the tile has more channels than Y, so there the row is
// part of the lane's offset.
struct StoreOffset {
    unsigned lane, scalar;
};
constexpr StoreOffset store_offset(bool whole, bool pixel, bool channel, unsigned first, unsigned row, unsigned oob) {
    return whole ? StoreOffset{pixel ? first : oob, row}
                 : StoreOffset{pixel && channel ? first + row : oob, 0};
}

}  // namespace xtc
