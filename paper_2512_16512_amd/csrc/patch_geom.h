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

}  // namespace xtc
