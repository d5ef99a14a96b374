// Record copies inside the encoder's launch (Sec. 4.4), for large snapshots:
// beside the workgroups that encode, the grid holds workgroups that copy the
// records of an earlier superblock (64 blocks) from their slots to the stream
// while later blocks are being encoded.  The encoder is bound by its
// instructions and LDS round trips, the copy by memory, so most of the copy
// disappears behind it.  Compression alone, cosmology 64M x 6: encoder 476 us
// and copy 131 us one after the other; now 490 us with the copies inside and
// 15 us for the rest.  Whole calls: 590 -> 519 us; LiDAR 20M x 3 with its range
// pass 222 -> 212; md 8M x 6 with decompression 170 -> 163; B = 512, 4M x 6
// 106 -> 100; float64 8M x 6 199 -> 190.
//
// Every workgroup is one wave.  The grid is laid out per XCD: workgroup g is
// taken to run on XCD g mod 8, and the workgroups of one XCD walk rows of one
// superblock each: 64 that encode its blocks and, from row place_delay
// on, kPlaceParts that copy the superblock encoded place_delay rows before.  A
// record is then written and read through the same XCD's L2, so its stores
// need no write-through (which cost the encoder 30 us at 64M x 6).  That
// placement is checked, not assumed: every block adds its XCD's number and its
// square to the superblock's word, and a superblock whose blocks did not all
// run on the copying wave's XCD is left to the copy kernel that follows, as
// are the last rows, whose copies would have nothing to hide behind.  Slots and
// lengths are read only after the whole superblock is there, and no two
// superblocks share a cache line of them (64 slots of whole 16-byte units), so
// no first-level cache holds an old copy.  The output buffer holds any stream of
// the shape (a rule of the launch), so nothing is checked against its size.
//
// A superblock's offset comes from a look-back over the words of those before
// it.  Every wait is bounded: a copying wave that has waited kPlaceSpins times,
// or meets a block left to the generic encoder, leaves its records to the copy
// kernel, so no result depends on the order in which the hardware starts
// workgroups, and a wave that waits for one that has not started goes on.
#pragma once

#include "gpz_internal.h"

namespace gpz {
namespace {

constexpr uint32_t kPlaceSpins = 2048;  // waits of about 1 us

// A superblock's word: record words, finished blocks, sum of their XCD
// numbers, sum of their squares, a block was left to the generic encoder, the
// offset is published.
constexpr int kSupCount = 28, kSupXcd = 36, kSupXcd2 = 47;
constexpr uint64_t kSupLeft = 1ull << 62, kSupKnown = 1ull << 63;

__device__ __forceinline__ uint64_t load_word(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t sup_words(uint64_t w) { return (uint32_t)w & 0xFFFFFFFu; }
__device__ __forceinline__ uint32_t sup_count(uint64_t w) {
    return (uint32_t)(w >> kSupCount) & 0xFFu;
}
// Number of the XCD this wave runs on (hardware register 20, bits 0-3).
__device__ __forceinline__ uint32_t xcd_id() {
    return (uint32_t)__builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11));
}

// Every store of this wave has reached its L2.
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The encoder's forms: the plain one, the few-blocks one, and the one whose
// launch also copies records (when a.sup is set).  Each is a kernel of its own:
// with one that looks at the arguments, a compression of 262k x 2 at B = 512
// took 23.1 us (22.5 plain, with the launches around it), 2.9M x 2 50.2 (49.5),
// 1M x 2 at B = 1024 26.8 (26.1).
enum Form : int { kPlain = 0, kFew = 1, kPlaces = 2 };

// Block b's record (len words) is in its slot.
template <int FORM>
__device__ __forceinline__ void finish_block(const EncodeArgs& a, uint32_t b, uint32_t len,
                                             uint32_t lane) {
    if (FORM == kPlaces && a.sup) {
        if (lane == 0) a.lens[b] = len;
        wait_stores();
        if (lane == 0) {
            const uint64_t x = xcd_id();
            __hip_atomic_fetch_add(a.sup + b / kSuper,
                                   (uint64_t)len | (1ull << kSupCount) | (x << kSupXcd) |
                                       (x * x << kSupXcd2),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    } else if (lane == 0) {
        a.lens[b] = len;
        if (FORM == kFew) a.defer[b] = 0u;
        else atomicAdd(&a.supsum[b / kSuper], len);  // order-independent sum
    }
}

// Leaves block b to the generic encoder (its record, length, superblock sum
// and permutation are all written there).
template <int FORM>
__device__ __forceinline__ void defer_block(const EncodeArgs& a, uint32_t b, uint32_t lane) {
    if (lane != 0) return;
    if (FORM == kFew) {
        a.defer[b] = 1u;
        return;
    }
    a.defer[atomicAdd(a.defer_count, 1u)] = b;
    if (FORM == kPlaces && a.sup)
        __hip_atomic_fetch_or(a.sup + b / kSuper, kSupLeft, __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
}

// What workgroup g of the encoder's grid does: encode block `block`, or copy
// part `part` of superblock `super`.
struct Role {
    bool encode, idle;
    uint32_t block, super, part;
};

__device__ __forceinline__ Role role_of(const EncodeArgs& a, uint32_t g) {
    if (!a.sup) return {true, false, g, 0u, 0u};
    constexpr uint32_t kRow = kSuper + kPlaceParts;
    const uint32_t delay = place_delay(a.B);
    const uint32_t x = g % kXcds, t = g / kXcds;
    Role r{};
    uint32_t row, i;
    if (t < delay * kSuper) {  // the first rows only encode
        row = t / kSuper;
        i = t % kSuper;
    } else {
        row = delay + (t - delay * kSuper) / kRow;
        i = (t - delay * kSuper) % kRow;
    }
    r.encode = i < kSuper;
    r.block = (row * kXcds + x) * kSuper + i;
    r.idle = r.encode && r.block >= a.nblocks;
    r.super = (row - delay) * kXcds + x;
    r.part = i - kSuper;
    return r;
}

typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kCopyLoads = 8;                       // 16-byte accesses of a lane and step
constexpr uint32_t kCopyWords = 256u * kCopyLoads;  // words of a step

// Words [k0, k0 + kCopyWords) of a record (len >= 4 words: the shortest holds
// two header words and two of its field).  Lanes past its
// end take its last four words again, so no access is predicated: the
// compiler counts exactly which loads a store has to wait for, and two records
// are in flight (with predicated stores it waited for every earlier store).
__device__ __forceinline__ uint32_t copy_word(uint32_t k0, int i, uint32_t len, uint32_t lane) {
    return min(k0 + 256u * (uint32_t)i + 4u * lane, len - 4u);
}
__device__ __forceinline__ void record_load(const uint32_t* src, uint32_t k0, uint32_t len,
                                            uint32_t lane, u32x4u (&v)[kCopyLoads]) {
    const uint8_t* const base = reinterpret_cast<const uint8_t*>(src);
#pragma unroll
    for (int i = 0; i < kCopyLoads; i++)
        v[i] = *reinterpret_cast<const u32x4u*>(base + 4u * copy_word(k0, i, len, lane));
}
__device__ __forceinline__ void record_store(uint32_t* dst, uint32_t k0, uint32_t len,
                                             uint32_t lane, const u32x4u (&v)[kCopyLoads]) {
    uint8_t* const base = reinterpret_cast<uint8_t*>(dst);
#pragma unroll
    for (int i = 0; i < kCopyLoads; i++)
        *reinterpret_cast<u32x4u*>(base + 4u * copy_word(k0, i, len, lane)) = v[i];
}

// Copies part `part` of the (whole) superblock s into the stream, with its
// records' length entries; part 0 also publishes the superblock's offset and
// writes its table entry.
__device__ __forceinline__ void place_records(const EncodeArgs& a, uint32_t s, uint32_t part,
                                              uint32_t lane) {
    const uint32_t first = s * kSuper;
    uint32_t spins = 0;
    uint64_t w;
    for (;;) {
        w = load_word(a.sup + s);
        if (w & kSupLeft) return;
        if (sup_count(w) == kSuper) break;
        if (++spins > kPlaceSpins) return;
        __builtin_amdgcn_s_sleep(4);
    }
    // every block ran on this XCD: 64 * sum(x^2) == (sum x)^2 only when all x
    // are the same
    const uint32_t sx = (uint32_t)(w >> kSupXcd) & 0x7FFu, sx2 = (uint32_t)(w >> kSupXcd2) & 0x7FFFu;
    if (sx != kSuper * xcd_id() || kSuper * sx2 != sx * sx) return;
    uint64_t off = 0;
    for (int top = (int)s - 1; top >= 0;) {
        const int p = top - (int)lane;
        const uint64_t v = p >= 0 ? load_word(a.sup + p) : kSupKnown;
        const uint64_t known = __ballot((v & kSupKnown) != 0);
        const uint64_t upto = known ? ((known & (~known + 1)) << 1) - 1 : ~0ull;
        if (__ballot((v & kSupLeft) != 0) & upto) return;
        if (__ballot(p >= 0 && sup_count(v) != kSuper) & upto) {
            if (++spins > kPlaceSpins) return;
            __builtin_amdgcn_s_sleep(4);
            continue;
        }
        uint64_t sum = p >= 0 && ((upto >> lane) & 1u) ? sup_words(v) : 0u;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o);
        off += sum;
        if (known) {
            const int k = top - (int)__builtin_ctzll(known);
            if (k >= 0) off += load_word(a.supoff + k);
            break;
        }
        top -= 64;
    }
    // (the compiler moves no read of a length or record above the waits)
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    asm volatile("" ::: "memory");
    const uint64_t lt_at = kHeaderWords + 2 * nsuper_of(a.nblocks) + a.F + first;
    const uint32_t len = a.lens[first + lane];
    const uint32_t start = wave_incl_scan_u32(len) - len;
    if (part == 0) {
        if (lane == 0)
            __hip_atomic_store(a.supoff + s, off, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        wait_stores();
        if (lane == 0)
            __hip_atomic_fetch_or(a.sup + s, kSupKnown, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    constexpr uint32_t kEach = kSuper / kPlaceParts;
    if (lane / kEach == part) a.out[lt_at + lane] = len;
    if (part == 0 && lane < 2) a.out[kHeaderWords + 2 * s + lane] = (uint32_t)(off >> (32 * lane));
    uint32_t* const recs = a.out + a.prefix + off;
    const uint32_t i0 = part * kEach;
    auto src = [&](uint32_t i) { return a.temp + (uint64_t)(first + i) * a.slot_words; };
    u32x4u va[kCopyLoads], vb[kCopyLoads];
    record_load(src(i0), 0, readlane(len, i0), lane, va);
#pragma unroll 1
    for (uint32_t i = i0; i < i0 + kEach; i += 2) {
        const uint32_t na = readlane(len, i), nb = readlane(len, i + 1);
        const uint32_t next = i + 2 < i0 + kEach ? i + 2 : i;
        record_load(src(i + 1), 0, nb, lane, vb);
        record_store(recs + readlane(start, i), 0, na, lane, va);
        record_load(src(next), 0, readlane(len, next), lane, va);
        record_store(recs + readlane(start, i + 1), 0, nb, lane, vb);
    }
    // records longer than a step
    if (__any(lane / kEach == part && len > kCopyWords)) {
#pragma unroll 1
        for (uint32_t i = i0; i < i0 + kEach; i++) {
            const uint32_t n = readlane(len, i);
            for (uint32_t k0 = kCopyWords; k0 < n; k0 += kCopyWords) {
                record_load(src(i), k0, n, lane, va);
                record_store(recs + readlane(start, i), k0, n, lane, va);
            }
        }
    }
    if (lane == 0) atomicOr(a.copied + s, 1u << part);
}

// Workgroups of the encoder's grid.
inline uint32_t encode_grid(const EncodeArgs& a) {
    return a.sup ? (uint32_t)placed_grid(a.nblocks, a.B) : a.nblocks;
}

}  // namespace
}  // namespace gpz
