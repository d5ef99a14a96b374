// The record copy (Sec. 4.4, step three), shared by the copy kernels and the
// few-blocks finish.
#pragma once

#include "gpz_internal.h"

namespace gpz {
namespace {

// Block b's record (len words) by one wave to its final offset off in the
// record area, with its length-table entry (and the superblock entry every 64
// blocks).
__device__ __forceinline__ void place_record(const CopyArgs& a, uint32_t b, uint32_t len,
                                             uint64_t off, uint32_t lane) {
    const uint64_t nsup = nsuper_of(a.nblocks);
    uint32_t* sup = a.out + kHeaderWords;
    uint32_t* lt = sup + 2 * nsup + a.F;
    uint32_t* recs = lt + a.nblocks;
    if (lane == 0) {
        lt[b] = len;
        if (b % kSuper == 0) {
            const uint32_t sb = b / kSuper;
            sup[2 * sb] = (uint32_t)(off & 0xFFFFFFFFu);
            sup[2 * sb + 1] = (uint32_t)(off >> 32);
        }
    }
    const uint32_t* src = a.temp + (uint64_t)b * a.slot_words;
    uint32_t* dst = recs + off;
    // 16 loads in flight per lane (4 KB per wave) before the stores; whole
    // 1024-word steps run without per-word predicates, at 32-bit offsets
    // from the scalar bases, and only the last step is predicated.
    constexpr int U = 16;
    const uint8_t* sb8 = reinterpret_cast<const uint8_t*>(src);
    uint8_t* db8 = reinterpret_cast<uint8_t*>(dst);
    const uint32_t whole = len & ~(64u * U - 1u);
    for (uint32_t k0 = 0; k0 < whole; k0 += 64 * U) {
        uint32_t v[U];
#pragma unroll
        for (int i = 0; i < U; i++)
            v[i] = __builtin_nontemporal_load(
                reinterpret_cast<const uint32_t*>(sb8 + 4u * (k0 + 64u * i + lane)));
#pragma unroll
        for (int i = 0; i < U; i++)
            *reinterpret_cast<uint32_t*>(db8 + 4u * (k0 + 64u * i + lane)) = v[i];
    }
    if (whole < len) {
        uint32_t v[U];
#pragma unroll
        for (int i = 0; i < U; i++) {
            const uint32_t k = whole + 64 * i + lane;
            v[i] = k < len ? __builtin_nontemporal_load(src + k) : 0u;
        }
#pragma unroll
        for (int i = 0; i < U; i++) {
            const uint32_t k = whole + 64 * i + lane;
            if (k < len) dst[k] = v[i];
        }
    }
}

}  // namespace
}  // namespace gpz
