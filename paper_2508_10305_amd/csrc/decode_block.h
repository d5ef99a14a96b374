// Pieces of the wave-per-block decoders (float32 in decode.hip, float64 in
// decode64.h): staging of packed arrays in LDS, extraction, location and
// checks of a block's record, expansion of its segment IDs.
#pragma once

#include "generic_block.h"

namespace gpz {
namespace {

template <int ITEMS>
__device__ __forceinline__ uint32_t pad_addr(uint32_t p) {
    return p + 4 * (p / ITEMS);
}

__device__ __forceinline__ bool eb_ok(float eb) {
    return __builtin_isfinite(eb) && eb >= 0x1p-120f && eb <= 0x1p120f;
}

// Copy `count` words (at most 64*L) from global memory into LDS with
// coalesced loads, all issued before the first LDS store, so the copy costs
// one memory round trip.  The number of 64-word steps selects a fully
// unrolled copy (a wave-uniform choice); inside the last step the lanes past
// the end load the array's last word again (so every load stays in bounds)
// and store it past the end, where the buffer still has room.  Offsets are
// 32-bit byte offsets from the array start, so each load takes the array's
// scalar base address and one offset register.
template <int N>
__device__ __forceinline__ void stage_steps(uint32_t* __restrict__ dst,
                                            const uint32_t* __restrict__ src, uint32_t count,
                                            uint32_t ln) {
    const uint8_t* b = reinterpret_cast<const uint8_t*>(src);
    uint32_t t[N];
#pragma unroll
    for (int u = 0; u < N; u++)
        t[u] = *reinterpret_cast<const uint32_t*>(b + 4u * min(ln + 64u * u, count - 1));
#pragma unroll
    for (int u = 0; u < N; u++) dst[ln + 64u * u] = t[u];
}

template <int N>
__device__ __forceinline__ void stage_pick(uint32_t steps, uint32_t* __restrict__ dst,
                                           const uint32_t* __restrict__ src, uint32_t count,
                                           uint32_t ln) {
    if constexpr (N > 0) {
        if (steps == N) stage_steps<N>(dst, src, count, ln);
        else stage_pick<N - 1>(steps, dst, src, count, ln);
    }
}

template <int L>
__device__ __forceinline__ void stage_words(uint32_t* __restrict__ dst,
                                            const uint32_t* __restrict__ src, uint32_t count,
                                            uint32_t lane) {
    if (count == 0) return;
    stage_pick<L>((count + 63) / 64, dst, src, count, lane);
}

// Value i of a fixed-length array of width w held in LDS (bits [i*w, i*w+w)).
__device__ __forceinline__ uint32_t extract(const uint32_t* __restrict__ words, uint32_t i,
                                            uint32_t w, uint32_t mask) {
    uint32_t bit = i * w;
    uint32_t wd = bit >> 5;
    uint32_t lo = words[wd], hi = words[wd + 1];
    return __builtin_amdgcn_alignbit(hi, lo, bit & 31u) & mask;
}

__device__ __forceinline__ uint32_t low_mask(uint32_t w) { return w >= 32u ? ~0u : ((1u << w) - 1u); }

// Sum over the wave of one 64-bit value per lane (every lane gets it).
__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// The first workgroup's copy of the stream's header for the host (the others
// do not wait for the pointer's load).
__device__ __forceinline__ void post_header(const DecodeArgs& a) {
    if (blockIdx.x != 0) return;
    if (a.header && threadIdx.x < kHeaderWords)
        a.header[threadIdx.x] = a.in[threadIdx.x];
}

// The stream as constant memory: no kernel writes it, and said so, a word at the
// same index for all lanes stays a scalar load (without, every one after the
// store that reports a bad record was a vector load).
typedef const uint32_t __attribute__((address_space(4))) StreamWord;
__device__ __forceinline__ const StreamWord* stream_words(const uint32_t* p) {
    return (const StreamWord*)(uintptr_t)p;
}

// Whether the stream's header is not that of the stream the caller asked for.
// `types`: the value-type flag asked for (0 float32, 1 float64); the wide-record
// flag beside it is free.  The words are the same for every lane: scalar loads.
__device__ __forceinline__ bool other_stream(const DecodeArgs& a, uint32_t types) {
    const StreamWord* h = stream_words(a.in);
    return ((h[0] ^ kMagic) | ((h[1] & ~(2u << 16)) ^ (kVersion | (types << 16))) |
            (h[2] ^ (uint32_t)(a.n & 0xFFFFFFFFu)) | (h[3] ^ (uint32_t)(a.n >> 32)) |
            (h[4] ^ a.F) | (h[5] ^ a.B) | (h[6] ^ (a.K | (a.KF << 8))) | (h[7] ^ a.nblocks)) != 0u;
}

// Whether the stream's eb table holds a bound out of range (every lane looks at
// a share of it; per-lane result).
__device__ __forceinline__ bool eb_table_bad(const DecodeArgs& a, uint32_t lane) {
    bool bad = false;
    const uint32_t* ebt = a.in + kHeaderWords + 2 * nsuper_of(a.nblocks);
    for (uint32_t f = lane; f < a.F; f += 64)
        if (!eb_ok(u2f(ebt[f]))) bad = true;
    return bad;
}

// The record of block b: false (and *a.err set) when the stream's header,
// tables or lengths are not those of the stream asked for.  A foreign header is
// reported by block 0 alone: a synchronous call starts with the decoder for the
// default parameters, whose every block finds one on any other stream, and the
// flag is then in host memory.  Its words are scalar loads beside the
// tables' and cost no round trip of their own (128M particles at B = 512: the
// whole call 306 us when the header came last and every block stored the flag,
// 287 now, 288 with the header fetched before any decoder runs; 285 when a
// block ended at the header, which cost every other stream 0.1 us).  The
// superblock entry is checked against the record area before anything is added
// to it, and the lengths are summed in 64 bits, so no sum can wrap and every
// accepted [rec, rec + len) lies inside the record area.
__device__ __forceinline__ bool locate_record(const DecodeArgs& a, uint32_t b, uint32_t lane,
                                              uint32_t types, const uint32_t*& rec,
                                              uint32_t& len) {
    const uint64_t nsup = nsuper_of(a.nblocks);
    const StreamWord* sup = stream_words(a.in) + kHeaderWords;
    const StreamWord* lens = sup + 2 * nsup + a.F;
    const uint64_t rec_total = a.in_words - a.prefix;
    const uint32_t sb = b / kSuper;
    const uint32_t first = sb * kSuper;
    const uint64_t sup_off = (uint64_t)sup[2 * sb] | ((uint64_t)sup[2 * sb + 1] << 32);
    const bool other = other_stream(a, types);
    const uint64_t mine = (first + lane < b) ? (uint64_t)lens[first + lane] : 0ull;
    const uint64_t sum = sup_off + wave_sum_u64(mine);
    // every lane holds the same sum: taken from lane 0 it is a scalar, and so
    // are the record pointer and every header word read through it
    const uint64_t off = ((uint64_t)readlane((uint32_t)(sum >> 32), 0) << 32) |
                         (uint64_t)readlane((uint32_t)sum, 0);
    len = lens[b];
    bool bad = sup_off > rec_total || off > rec_total || (uint64_t)len > rec_total - off;
    if (b == 0 && (sup[0] | sup[1]) != 0u) bad = true;
    if (a.exact && b + 1 == a.nblocks && off + len != rec_total) bad = true;
    if (eb_table_bad(a, lane)) bad = true;
    if (b == first && sb > 0) {
        // consistency of this superblock's offset with the previous one
        const uint64_t pl = lens[first - kSuper + lane];
        const uint64_t prev = ((uint64_t)sup[2 * sb - 2] | ((uint64_t)sup[2 * sb - 1] << 32));
        if (prev > rec_total || prev + wave_sum_u64(pl) != off) bad = true;
    }
    if (other || __any(bad)) {
        if (lane == 0 && (b == 0 || !other)) *a.err = 1u;
        return false;
    }
    rec = a.in + a.prefix + off;
    return true;
}

// Undoes the delta and run-length coding (Sec. 4.3) of a record's segment IDs
// (U runs, gaps then counts from rec + 2): every position's ID ends up in
// `buf` in the padded blocked layout.  False when the IDs or the run lengths
// do not fit the block.  STEPS 0: the record is in LDS already (`rec`, beside
// `buf`).
template <int ITEMS, int STEPS>
__device__ __forceinline__ bool expand_runs(const uint32_t* rec, uint32_t U, uint32_t w_gap,
                                            uint32_t w_cnt, uint32_t gw, uint32_t cw, uint32_t nb,
                                            uint32_t keybits, uint32_t lane, uint32_t* buf) {
    constexpr uint32_t B = 64 * ITEMS;
    constexpr uint32_t G = ITEMS / 4;
    const uint32_t* words = STEPS ? buf : rec + 2;
    uint32_t* keys = buf;
    if constexpr (STEPS > 0) {
        stage_words<STEPS>(buf, rec + 2, gw + cw, lane);
        wave_lds_sync();
    }
    uint32_t g1[ITEMS], c1[ITEMS];
    uint32_t gs = 0, cs = 0;
    {
        const uint32_t gm = low_mask(w_gap), cm = low_mask(w_cnt);
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            uint32_t i = lane * ITEMS + j;
            g1[j] = i < U ? extract(words, i, w_gap, gm) + 1u : 0u;
            c1[j] = i < U ? extract(words + gw, i, w_cnt, cm) + 1u : 0u;
            gs += g1[j];
            cs += c1[j];
        }
    }
    const uint32_t gincl = wave_incl_scan_u32(gs), cincl = wave_incl_scan_u32(cs);
    const uint32_t gtot = (uint32_t)__shfl((int)gincl, 63), ctot = (uint32_t)__shfl((int)cincl, 63);
    // largest ID = sum(gap+1) - 1 must fit K*KF bits; run lengths sum to nb
    if (ctot != nb || gtot == 0 || gtot - 1u >= (1u << keybits)) {
        return false;
    }
    // mark run starts with their ID; IDs increase with position, so a prefix
    // maximum over positions gives every position its ID
    wave_lds_sync();  // the packed gaps and counts are read; `keys` reuses them
    for (uint32_t p = lane; p < B; p += 64) keys[pad_addr<ITEMS>(p)] = 0u;
    wave_lds_sync();
    {
        uint32_t u = gincl - gs, st = cincl - cs;
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            uint32_t i = lane * ITEMS + j;
            if (i < U) {
                u += g1[j];
                keys[pad_addr<ITEMS>(st)] = u - 1u;
                st += c1[j];
            }
        }
    }
    wave_lds_sync();
    {
        uint32_t key[ITEMS];
        uint32_t run = 0;
        const uint4* kb = reinterpret_cast<const uint4*>(keys + lane * (ITEMS + 4));
#pragma unroll
        for (int g = 0; g < G; g++) {
            uint4 t = kb[g];
            run = max(run, t.x);
            key[4 * g + 0] = run;
            run = max(run, t.y);
            key[4 * g + 1] = run;
            run = max(run, t.z);
            key[4 * g + 2] = run;
            run = max(run, t.w);
            key[4 * g + 3] = run;
        }
        uint32_t carry = wave_incl_max_u32(run);
        carry = (uint32_t)__shfl_up((int)carry, 1);
        if (lane == 0) carry = 0;
        wave_lds_sync();
        uint4* kw = reinterpret_cast<uint4*>(keys + lane * (ITEMS + 4));
#pragma unroll
        for (int g = 0; g < G; g++)
            kw[g] = make_uint4(max(key[4 * g], carry), max(key[4 * g + 1], carry),
                               max(key[4 * g + 2], carry), max(key[4 * g + 3], carry));
    }
    wave_lds_sync();
    return true;
}

}  // namespace
}  // namespace gpz
