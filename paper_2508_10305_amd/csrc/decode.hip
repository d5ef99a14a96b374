// Block decoder (Sec. 3.2: decompression reverses the compression steps,
// without un-sorting): one wave64 per block locates its record through the
// superblock table, undoes the delta and run-length coding of the segment
// IDs, unpacks the fixed-length payloads, rebuilds every value with
// fma(q, 2eb, lo), patches outliers and stores the block in sorted order.
//
// Each coded array is first copied into LDS with coalesced loads; values are
// then extracted from LDS.  Outputs are written "striped": lane l produces
// positions 256k + 4l + {0..3}, so one 16-byte store per lane covers 1 KB of
// contiguous output per instruction.  One wave per workgroup: LDS traffic
// between its lanes is ordered by wave_lds_sync().  Every read of the record
// is checked against its length first; a malformed record sets the error
// flag and the block is skipped.
#include "decode64.h"
#include "decode_block.h"
#include "decode_layout.h"

namespace gpz {
namespace {

template <int ITEMS>
struct DecodeSmem {
    static constexpr uint32_t B = 64 * ITEMS;
    // widest coded arrays: payload 24 bits/value; gaps 15 + counts 12 bits
    static constexpr uint32_t kPay = (B * 24) / 32 + 2;
    static constexpr uint32_t kRle = (B * 15) / 32 + (B * 12) / 32 + 4;
    static constexpr uint32_t kWords = ((kPay > kRle ? kPay : kRle) + 3) & ~3u;  // 16-byte multiple
    static constexpr uint32_t kPadB = 64 * (ITEMS + 4);
    // The packed words, the key expansion and the outlier staging are never
    // live at the same time: one region serves all three (barriers between
    // the phases), which keeps the workgroup's LDS small enough for high
    // occupancy.
    static constexpr uint32_t kA = kWords > kPadB ? kWords : kPadB;
    static constexpr uint32_t kBuf = kA > B ? kA : B;
    // 64-word steps of the widest array, which stage_words fills whole
    static constexpr int kSteps = (int)((kWords + 63) / 64);
    static_assert(64 * kSteps <= kBuf, "staged steps stay inside buf");
    uint32_t buf[kBuf];
};

// The decoder's LDS: its own buffer, or the generic record decoder's when a
// record holds a field coded with 64-bit steps.
template <int ITEMS>
union DecodeShared {
    DecodeSmem<ITEMS> fast;
    GenDecodeSmem<64 * ITEMS> wide;
};

// WAVES > 1: the record is first copied to `recbuf` in LDS by all waves, in one
// memory round trip for up to kFewRecWords words, and decoded from there, wave w
// taking fields w, w + WAVES, ... with an LDS region of its own; a longer
// coded record is decoded by wave 0 as without.  For snapshots of few blocks, where
// the time is one block's chain of round trips (tables, header, runs, and two
// for every field) and of instructions, not the bytes.
template <int ITEMS, uint32_t WAVES = 1>
__device__ __forceinline__ void decode_block(const DecodeArgs& a, uint32_t b,
                                             DecodeShared<ITEMS>& shared,
                                             DecodeShared<ITEMS>* own = nullptr,
                                             uint32_t* recbuf = nullptr) {
    constexpr bool WHOLE = WAVES > 1;
    const uint32_t wave =
        WHOLE ? (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0u;
    DecodeSmem<ITEMS>& sm = WHOLE ? own[wave].fast : shared.fast;
    constexpr uint32_t B = 64 * ITEMS;
    constexpr uint32_t G = ITEMS / 4;  // 16-byte groups per lane
    uint32_t* const keys = sm.buf;
    uint32_t* const ystage = sm.buf;

    const uint32_t lane = WHOLE ? threadIdx.x & 63u : threadIdx.x;
    const uint64_t base = (uint64_t)b * B;
    const uint32_t nb = (uint32_t)((a.n - base) < B ? (a.n - base) : B);
    const uint32_t F = a.F, K = a.K, KF = a.KF;
    const uint32_t* ebt = a.in + kHeaderWords + 2 * nsuper_of(a.nblocks);
    const uint32_t* rec;
    uint32_t len;
    if (!locate_record(a, b, lane, 0u, rec, len)) return;
    bool in_lds = false;
    if constexpr (WHOLE) {
        // (every wave has located the same record: what follows is uniform)
        len = readlane(len, 0);
        in_lds = len <= kFewRecWords;
        if (in_lds) {
            constexpr uint32_t kStep = 1024;
            static_assert(kFewRecWords % kStep == 0, "whole staging steps stay inside the buffer");
            for (uint32_t k = kStep * wave; k < len; k += kStep * WAVES)
                stage_words<kStep / 64>(recbuf + k, rec + k, min(len - k, kStep), lane);
            __syncthreads();
        }
    }
    // Word k of the record.  Through a 64-bit index, as the record's other
    // addresses: with a 32-bit one their reads shared no address, and the decoder
    // of 1.3M particles x 6 took 18.9 us instead of 18.3.  At B = 2048 the 32-bit
    // index leaves 127 registers instead of 136, four waves per SIMD instead of
    // three: 32M particles x 2 106 us instead of 124 (whole call).
    auto word = [&](uint64_t k) -> uint32_t {
        if constexpr (WHOLE) return (uint32_t)__builtin_amdgcn_readfirstlane((int)recbuf[(uint32_t)k]);
        else if constexpr (ITEMS == 32) return stream_words(rec)[(uint32_t)k];
        else return stream_words(rec)[k];
    };
    const uint32_t h0 = len == 0 ? 0u : WHOLE && !in_lds ? rec[0] : word(0);
    const uint32_t mode = h0 & 3u;

    if (len != 0 && mode == 0 && (h0 >> 31)) {
        // a field coded with 64-bit steps (Sec. 5.3): the generic record
        // decoder, run by this wave, when the header announces such records
        // (corrupt otherwise)
        if (!((a.in[1] >> 17) & 1u)) {
            if (lane == 0) *a.err = 1u;
            return;
        }
        gen_decode_record<64 * ITEMS, 64 * WAVES, false>(a, b, rec, len, shared.wide);
        return;
    }
    if (len == 0 || mode > 1) {
        if (lane == 0) *a.err = 1u;
        return;
    }
    if (mode == 1) {
        if (h0 != 1u || len != 1 + F * nb) {
            if (lane == 0) *a.err = 1u;
            return;
        }
        for (uint32_t f = 0; f < F; f++) {
            float* yf = a.y[f] + base;
            const uint32_t* src = rec + 1 + f * nb;
            for (uint32_t i = 64 * wave + lane; i < nb; i += 64 * WAVES) yf[i] = u2f(src[i]);
        }
        return;
    }

    if constexpr (WHOLE) {
        // a coded record too long for the LDS, with 32-bit steps only: one wave
        if (!in_lds) {
            if (wave == 0) decode_block<ITEMS, 1>(a, b, shared);
            return;
        }
    }

    // ---- coded record header
    const uint32_t U = h0 >> 2;
    const uint32_t h1 = len > 1 ? word(1) : 0xFFFFFFFFu;
    const uint32_t w_gap = h1 & 31u, w_cnt = (h1 >> 5) & 31u;
    const uint32_t s0 = (h1 >> 10) & 31u, s1 = (h1 >> 15) & 31u, s2 = (h1 >> 20) & 31u;
    bool bad = len < 2 || (h1 >> 25) != 0u || U < 1 || U > nb || w_gap > 15 || w_cnt > 12;
    bad |= (KF < 2 && s1 != 0) || (KF < 3 && s2 != 0);
    bad |= (s0 + K > 24) || (KF > 1 && s1 + K > 24) || (KF > 2 && s2 + K > 24);
    const uint32_t gw = words_for(U, w_gap), cw = words_for(U, w_cnt);
    bad |= (uint64_t)2 + gw + cw > len;
    if (bad) {
        if (lane == 0) *a.err = 1u;
        return;
    }

    // ---- undo delta + run-length coding (Sec. 4.3)
    if (!expand_runs<ITEMS, WHOLE ? 0 : DecodeSmem<ITEMS>::kSteps>(
            WHOLE ? recbuf : rec, U, w_gap, w_cnt, gw, cw, nb, K * KF, lane, sm.buf)) {
        if (lane == 0) *a.err = 1u;
        return;
    }
    // striped positions of this lane: p = 256 g + 4 lane + e
    uint32_t skey[ITEMS];
#pragma unroll
    for (int g = 0; g < G; g++)
#pragma unroll
        for (int e = 0; e < 4; e++) skey[4 * g + e] = keys[pad_addr<ITEMS>(256 * g + 4 * lane + e)];

    // ---- fields
    uint64_t pos = 2 + gw + cw;
    const bool full = nb == B;
    for (uint32_t f = 0; f < F; f++) {
        if (pos + 2 > len) {
            bad = true;
            break;
        }
        const float lo = u2f(word(pos));
        const uint32_t wn = word(pos + 1);
        const uint32_t w = wn & 31u, nout = wn >> 5;
        uint32_t s = 0, shift = 0;
        if (f < KF) {
            s = f == 0 ? s0 : (f == 1 ? s1 : s2);
            shift = K * (KF - 1 - f);
        }
        const uint32_t wlim = f < KF ? s : 24u;
        const uint32_t pw = words_for(nb, w);
        if (w > wlim || nout > nb || pos + 2 + pw + 2 * (uint64_t)nout > len) {
            bad = true;
            break;
        }
        if (WHOLE && f % WAVES != wave) {
            pos += 2 + pw + 2 * (uint64_t)nout;
            continue;
        }
        const float twoeb = 2.0f * u2f(ebt[f]);
        wave_lds_sync();  // previous users of the buffer are done
        const uint32_t* words = sm.buf;
        if constexpr (WHOLE) {
            words = recbuf + pos + 2;
        } else {
            stage_words<DecodeSmem<ITEMS>::kSteps>(sm.buf, rec + pos + 2, pw, lane);
            wave_lds_sync();
        }
        const uint32_t mask = low_mask(w);
        uint32_t y[ITEMS];
        if (f < KF) {
            // a key field's code: the position's segment (its K bits of the
            // ID) above the s stored offset bits
#pragma unroll
            for (int g = 0; g < G; g++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const uint32_t p = 256 * g + 4 * lane + e;
                    const uint32_t v = extract(words, p, w, mask);
                    const uint32_t q = (__builtin_amdgcn_ubfe(skey[4 * g + e], shift, K) << s) | v;
                    y[4 * g + e] = f2u(__builtin_fmaf((float)q, twoeb, lo));
                }
        } else {
#pragma unroll
            for (int g = 0; g < G; g++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const uint32_t p = 256 * g + 4 * lane + e;
                    const uint32_t v = extract(words, p, w, mask);
                    y[4 * g + e] = f2u(__builtin_fmaf((float)v, twoeb, lo));
                }
        }
        if (nout) {
            // patch outliers through LDS (the staging reuses `words`)
            const uint32_t* ol = (WHOLE ? recbuf : rec) + pos + 2 + pw;
            wave_lds_sync();
#pragma unroll
            for (int g = 0; g < G; g++)
                reinterpret_cast<uint4*>(ystage)[64 * g + lane] =
                    make_uint4(y[4 * g], y[4 * g + 1], y[4 * g + 2], y[4 * g + 3]);
            wave_lds_sync();
            bool obad = false;
            for (uint32_t k = lane; k < nout; k += 64) {
                uint32_t op = ol[2 * k];
                uint32_t prevp = k ? ol[2 * k - 2] : 0u;
                if (op >= nb || (k && prevp >= op)) obad = true;
                else ystage[op] = ol[2 * k + 1];
            }
            if (__any(obad)) {
                bad = true;
                break;
            }
            wave_lds_sync();
#pragma unroll
            for (int g = 0; g < G; g++) {
                uint4 t = reinterpret_cast<const uint4*>(ystage)[64 * g + lane];
                y[4 * g] = t.x;
                y[4 * g + 1] = t.y;
                y[4 * g + 2] = t.z;
                y[4 * g + 3] = t.w;
            }
        }
        float* yf = a.y[f] + base;
        if (full && ((reinterpret_cast<uintptr_t>(a.y[f].get()) & 15u) == 0)) {
#pragma unroll
            for (int g = 0; g < G; g++) {
                u32x4 t = {y[4 * g], y[4 * g + 1], y[4 * g + 2], y[4 * g + 3]};
                __builtin_nontemporal_store(t, reinterpret_cast<u32x4*>(yf + 256 * g + 4 * lane));
            }
        } else {
#pragma unroll
            for (int g = 0; g < G; g++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const uint32_t p = 256 * g + 4 * lane + e;
                    if (p < nb) yf[p] = u2f(y[4 * g + e]);
                }
        }
        pos += 2 + pw + 2 * (uint64_t)nout;
    }
    if (bad || pos != len) {
        if (lane == 0) *a.err = 1u;
    }
}

template <int ITEMS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(8))) void decode_blocks(DecodeArgs a) {
    __shared__ __align__(16) DecodeShared<ITEMS> sm;
    decode_block<ITEMS>(a, blockIdx.x, sm);
    post_header(a);
}

// The same for a snapshot of few blocks (few_blocks_per_cu: as many as are
// resident at once): four waves a block.  B = 1024, 6 fields, event
// pair included: 10k particles 18.4 -> 12.6 us, 524k 18.8 -> 13.8, 1M
// 20.5 -> 16.2 (with one wave and the record in LDS 15.3, 16.0 and 16.8);
// above, the bytes begin to count and eight blocks per SIMD are faster.
constexpr uint32_t kFewWaves = 4;

template <int ITEMS>
__global__ __launch_bounds__(64 * kFewWaves) void decode_few(DecodeArgs a) {
    __shared__ __align__(16) DecodeShared<ITEMS> own[kFewWaves];
    __shared__ __align__(16) uint32_t recbuf[few_rec_room(64 * ITEMS)];
    static_assert(sizeof(own[0]) % 16 == 0, "every wave's region is stored 16 bytes at a time");
    static_assert((sizeof(own) + sizeof(recbuf)) * few_blocks_per_cu(64 * ITEMS, 1) <= 160 * 1024,
                  "the blocks of the form share a CU's LDS");
    decode_block<ITEMS, kFewWaves>(a, blockIdx.x, own[0], own, recbuf);
    post_header(a);
}

// Persistent decoder over the blocks of many streams: each wave takes `tile`
// consecutive blocks from a device work queue until the queue is empty.
template <int ITEMS>
__global__ __launch_bounds__(64) void decode_batch(const DecodeArgs* __restrict__ jobs,
                                                   const BatchLaunch* __restrict__ L) {
    __shared__ __align__(16) DecodeShared<ITEMS> sm;
    const uint32_t total = L->total_blocks, njobs = L->njobs, tile = L->tile;
    const uint32_t* prefix = L->block_prefix;
    for (;;) {
        uint32_t item = 0;
        if (threadIdx.x == 0) item = atomicAdd(L->counter + 1, tile);
        item = (uint32_t)__builtin_amdgcn_readfirstlane((int)item);
        if (item >= total) break;
        const uint32_t end = min(item + tile, total);
        for (uint32_t g = item; g < end; g++) {
            const uint32_t j = find_job(prefix, njobs, g);
            decode_block<ITEMS>(jobs[j], g - prefix[j], sm);
            __syncthreads();
        }
    }
}

// Direct form of decode_batch: one workgroup per block of the batch's
// capacity (no loop around the block, so a smaller register budget).  At
// B = 1024 seven waves per SIMD, not eight: eight leaves 63 registers and 29
// scalars spilled into them (24 snapshots, 16M particles x 6, both
// directions: 337 us at eight, 334 at seven).
template <int ITEMS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(ITEMS == 32 ? 3 : ITEMS == 16 ? 7 : 8))) void decode_batch_direct(const DecodeArgs* __restrict__ jobs,
                                                          const BatchLaunch* __restrict__ L) {
    __shared__ __align__(16) DecodeShared<ITEMS> sm;
    const uint32_t g = blockIdx.x;
    if (g >= L->total_blocks) return;
    const uint32_t* prefix = L->block_prefix;
    const uint32_t j = find_job(prefix, L->njobs, g);
    decode_block<ITEMS>(jobs[j], g - prefix[j], sm);
}

// A stream of a snapshot with no particles holds only its header, its
// superblock table (empty) and its eb table: one wave checks them, so the
// caller needs no host copy of the stream.
__global__ __launch_bounds__(64) void check_empty_stream(DecodeArgs a) {
    const uint32_t lane = threadIdx.x;
    bool bad = other_stream(a, 0u) || eb_table_bad(a, lane);
    if (a.exact && a.in_words != a.prefix) bad = true;
    if (__any(bad) && lane == 0) *a.err = 1u;
}

}  // namespace

hipError_t launch_decode_batch(const DecodeArgs* jobs, const BatchLaunch* L,
                               const BatchShape& S, hipStream_t s) {
    dim3 block(64);
    if (S.grid) {
        dim3 grid(S.grid);
        switch (S.B) {
            case 256: hipLaunchKernelGGL(decode_batch<4>, grid, block, 0, s, jobs, L); break;
            case 512: hipLaunchKernelGGL(decode_batch<8>, grid, block, 0, s, jobs, L); break;
            case 1024: hipLaunchKernelGGL(decode_batch<16>, grid, block, 0, s, jobs, L); break;
            case 2048: hipLaunchKernelGGL(decode_batch<32>, grid, block, 0, s, jobs, L); break;
            default: return hipErrorInvalidValue;
        }
    } else {
        dim3 grid(S.direct_grid);
        switch (S.B) {
            case 256: hipLaunchKernelGGL(decode_batch_direct<4>, grid, block, 0, s, jobs, L); break;
            case 512: hipLaunchKernelGGL(decode_batch_direct<8>, grid, block, 0, s, jobs, L); break;
            case 1024: hipLaunchKernelGGL(decode_batch_direct<16>, grid, block, 0, s, jobs, L); break;
            case 2048: hipLaunchKernelGGL(decode_batch_direct<32>, grid, block, 0, s, jobs, L); break;
            default: return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

hipError_t launch_decode(const DecodeArgs& a, hipStream_t s) {
    if (a.nblocks == 0) {
        hipLaunchKernelGGL(check_empty_stream, dim3(1), dim3(64), 0, s, a);
        return hipGetLastError();
    }
    dim3 grid(a.nblocks), block(64);
    if (a.nblocks <= few_blocks_per_cu(a.B, a.F) * device_cu_count()) {
        const dim3 few(64 * kFewWaves);
        switch (a.B) {
            case 256: hipLaunchKernelGGL(decode_few<4>, grid, few, 0, s, a); break;
            case 512: hipLaunchKernelGGL(decode_few<8>, grid, few, 0, s, a); break;
            case 1024: hipLaunchKernelGGL(decode_few<16>, grid, few, 0, s, a); break;
            case 2048: hipLaunchKernelGGL(decode_few<32>, grid, few, 0, s, a); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    switch (a.B) {
        case 256: hipLaunchKernelGGL(decode_blocks<4>, grid, block, 0, s, a); break;
        case 512: hipLaunchKernelGGL(decode_blocks<8>, grid, block, 0, s, a); break;
        case 1024: hipLaunchKernelGGL(decode_blocks<16>, grid, block, 0, s, a); break;
        case 2048: hipLaunchKernelGGL(decode_blocks<32>, grid, block, 0, s, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_decode64(const DecodeArgs& a, hipStream_t s) {
    if (a.B != 1024u) return hipErrorInvalidValue;
    if (a.nblocks == 0) return hipSuccess;
    hipLaunchKernelGGL(decode_blocks64, dim3(a.nblocks), dim3(64), 0, s, a);
    return hipGetLastError();
}

}  // namespace gpz
