// The LDS of a wave of the short-row kernels (prune_short.hip), in plain C++ so that it can be checked on the host.
//
// 64 / G rows lie there as they lie in the tensor, the output slots behind them.  The G lanes of a row have parts of
// ceil(cols / G) entries; those of the last lanes may be shorter, or begin past the row's end.  Every lane reads as many
// entries as the longest part has, in whole blocks, and does not use those that are not its own: in the last row these
// lie behind the rows.
#pragma once
#include <cstddef>

namespace slimfit {

constexpr int kShortHeldBlock = 4;          // entries a block where a lane's part is held in registers; elsewhere one

// entries past a row's end that its last lane reads
constexpr int short_entries_past(int cols, int G, int block)
{
    const int part = (cols + G - 1) / G;
    return (G - 1) * part + (part + block - 1) / block * block - cols;
}
constexpr size_t short_rows_bytes(int cols, int G, int element_bytes)
{
    return (size_t)(64 / G * cols * element_bytes + 15) / 16 * 16;
}
// the launch's dynamic LDS: the rows, then the output slots or what is read there, whichever is more
constexpr size_t short_lds_bytes(int cols, int k, int G, int element_bytes, int block)
{
    const size_t slots = (size_t)(64 / G) * (size_t)k * 4, past = (size_t)(short_entries_past(cols, G, block) * element_bytes + 15) / 16 * 16;
    return short_rows_bytes(cols, G, element_bytes) + (slots > past ? slots : past);
}

}  // namespace slimfit
