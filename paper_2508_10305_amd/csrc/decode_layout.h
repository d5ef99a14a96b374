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

}  // namespace gpz
