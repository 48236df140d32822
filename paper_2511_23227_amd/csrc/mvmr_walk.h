// How a wave walks the triplet list, in code that runs on the host too; not part of the C ABI.
#pragma once

#include <stdint.h>

#include <hip/hip_runtime.h>

namespace pcpp {

// Byte offset of word `first + lane_word` of an index array, for the offset operand of a buffer load.  Requests run ahead
// of the work, past the end of the list, and the descriptor must reject those: it compares this operand with the array's
// size, while an address part in the scalar offset operand may not take part in the comparison.  So the whole offset goes
// here.  It cannot wrap: lists have fewer than 2^30 - 1023 words (MAX_BUFFER_BYTES), and the walk below asks for no word
// more than 286 behind the last one.
__host__ __device__ inline uint32_t index_offset(uint32_t first, uint32_t lane_word) { return (first + lane_word) * 4u; }

// A wave's batches of the weight gradient: position in the chunk, end of its cell's run inside the chunk, the cell.  The
// waves of a block take a run's batches in turn; a batch never crosses the end of a run.
struct BatchCursor { uint32_t pos, end; int k; };

// The first batch at or behind `start` of c's run, or, past its end, of a later one (`own`: the wave's first position in a
// run).  Behind the chunk's last run the position stays past `p_end`: such a batch has no triplets.
template <typename EndOf>
__host__ __device__ inline void settle_batch(BatchCursor &c, uint32_t start, uint32_t p_end, uint32_t own, EndOf end_of)
{
    c.pos = start;
    while (c.pos >= c.end && c.end < p_end) {
        const uint32_t s = c.end;
        ++c.k;
        c.end = end_of(c.k);
        c.pos = s + own;
    }
}

}  // namespace pcpp
