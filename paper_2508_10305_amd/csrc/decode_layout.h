// Sizes of the few-blocks decoder's LDS (decode.hip).  Plain constants, so
// that they can be checked on the host against the streams themselves.
#pragma once

#include <stdint.h>

namespace gpz {

// Words of the longest record that is decoded from LDS.
constexpr uint32_t kFewRecWords = 4096;

// Words of the buffer that holds it, for blocks of B values.  An array is
// extracted at all B positions, also in a partial block whose array is
// shorter, so the reads of a record's last array run past the record's end:
// up to B values of 24 bits and the second word of the last one.
constexpr uint32_t few_rec_room(uint32_t B) { return kFewRecWords + B * 24 / 32 + 2; }

// Blocks per CU up to which a snapshot is decoded in that form (0: never).
// Every workgroup has to be resident at once: a block takes 40 KB of the CU's
// 160 at B = 1024 and 59 KB at 2048, and a second round costs more than the form
// gains (B = 2048, 3 fields, 768 blocks: 18.8 us with one wave a block, 25.4 as
// three blocks per CU).  At B = 2048 a record of more than four fields is usually
// longer than kFewRecWords (6 fields of 13 bits: 5000 words), and one wave then
// decodes it after the others have looked at it: 22.5 us with one wave a block
// against 24.2 at 16 blocks; with 3 fields 17.6 against 14.5.  Below, long
// records lose nothing (B = 1024, 64 fields, 10 blocks: 90.5 and 80.9).
constexpr uint32_t few_blocks_per_cu(uint32_t B, uint32_t F) {
    return B <= 1024 ? 4u : F <= 4 ? 2u : 0u;
}

}  // namespace gpz
