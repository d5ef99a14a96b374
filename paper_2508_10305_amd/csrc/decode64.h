// Block decoder for float64 streams at B = 1024: one wave64 per block, as
// decode.hip does for float32 streams.  A field's packed values (up to 53 bits)
// are staged in LDS with coalesced loads and extracted from there; each store
// instruction covers 1 KB of contiguous output (lane l holds positions
// 128k + 2l + {0, 1}).
//
// What bounds it: the output's write (8 bytes a value); the staging buffer of
// 7 KB lets five waves share a SIMD.  The whole call on 8M x 6: 276 us with
// the generic decoder (one lane per 4 positions, each reading its bits from
// memory), 125 here, of which about 45 are the call's launches and waits;
// with every field on 64-bit steps 323 -> 159.
#pragma once

#include "decode_block.h"

namespace gpz {
namespace {

constexpr int kItems = 16;
constexpr uint32_t kB = 64 * kItems;
// LDS words: the widest payload (1024 values of 53 bits) and the words an
// extraction may touch past it, in whole 64-word steps; the segment IDs in the
// padded blocked layout use the same region.
constexpr int kSteps64 = (int)((kB * 53 / 32 + 2 + 63) / 64);
constexpr uint32_t kBuf64 = 64 * kSteps64;
static_assert(kBuf64 >= 64 * (kItems + 4), "the padded IDs fit the region");

typedef double f64x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void decode_block64(const DecodeArgs& a, uint32_t b, uint32_t* words) {
    const uint32_t lane = threadIdx.x;
    const uint64_t base = (uint64_t)b * kB;
    const uint32_t nb = (uint32_t)((a.n - base) < kB ? (a.n - base) : kB);
    const uint32_t F = a.F, K = a.K, KF = a.KF;
    const uint32_t* ebt = a.in + kHeaderWords + 2 * nsuper_of(a.nblocks);
    const uint32_t* rec;
    uint32_t len;
    if (!locate_record(a, b, lane, 1u, rec, len)) return;
    const uint32_t h0 = len ? rec[0] : 0u;
    const uint32_t mode = h0 & 3u;
    if (len == 0 || mode > 1) {
        if (lane == 0) *a.err = 1u;
        return;
    }
    if (mode == 1) {
        if (h0 != 1u || len != 1 + 2 * F * nb) {
            if (lane == 0) *a.err = 1u;
            return;
        }
        for (uint32_t f = 0; f < F; f++) {
            uint64_t* yf = reinterpret_cast<uint64_t*>(a.y[f].get()) + base;
            const uint32_t* src = rec + 1 + 2 * f * nb;
            for (uint32_t i = lane; i < nb; i += 64)
                yf[i] = (uint64_t)src[2 * i] | ((uint64_t)src[2 * i + 1] << 32);
        }
        return;
    }

    // ---- coded record header
    const uint32_t U = (h0 & 0x7FFFFFFFu) >> 2, any_wide = h0 >> 31;
    const uint32_t h1 = len > 1 ? rec[1] : 0xFFFFFFFFu;
    const uint32_t w_gap = h1 & 31u, w_cnt = (h1 >> 5) & 31u;
    const uint32_t s0 = ((h1 >> 10) & 31u) | (((h1 >> 25) & 1u) << 5);
    const uint32_t s1 = ((h1 >> 15) & 31u) | (((h1 >> 26) & 1u) << 5);
    const uint32_t s2 = ((h1 >> 20) & 31u) | (((h1 >> 27) & 1u) << 5);
    bool bad = len < 2 || (h1 >> 28) != 0u || U < 1 || U > nb || w_gap > 15 || w_cnt > 12;
    // a wide record in a stream whose header does not announce one
    bad |= any_wide && !((a.in[1] >> 17) & 1u);
    bad |= (KF < 2 && s1 != 0) || (KF < 3 && s2 != 0);
    bad |= (s0 + K > 53) || (KF > 1 && s1 + K > 53) || (KF > 2 && s2 + K > 53);
    const uint32_t gw = words_for(U, w_gap), cw = words_for(U, w_cnt);
    bad |= (uint64_t)2 + gw + cw > len;
    if (bad) {
        if (lane == 0) *a.err = 1u;
        return;
    }
    if (!expand_runs<kItems, kSteps64>(rec, U, w_gap, w_cnt, gw, cw, nb, K * KF, lane, words)) {
        if (lane == 0) *a.err = 1u;
        return;
    }
    // positions of this lane: 128 k + 2 lane + e; their IDs (at most 15 bits),
    // two to a register
    uint32_t skey[kItems / 2];
#pragma unroll
    for (int k = 0; k < kItems / 2; k++) {
        const uint32_t at = pad_addr<kItems>(128 * k + 2 * lane);
        skey[k] = words[at] | (words[at + 1] << 16);
    }

    // ---- fields
    uint64_t pos = 2 + gw + cw;
    uint32_t seen_wide = 0;
    const bool full = nb == kB;
#pragma unroll 1
    for (uint32_t f = 0; f < F; f++) {
        if (pos + 3 > len) {
            bad = true;
            break;
        }
        const double lo = u2d((uint64_t)rec[pos] | ((uint64_t)rec[pos + 1] << 32));
        const uint32_t wn = rec[pos + 2];
        const bool wide = (wn >> 31) != 0;
        const uint32_t w = wide ? (wn & 63u) : (wn & 31u);
        const uint32_t nout = wide ? ((wn >> 6) & 0x1FFFFFFu) : ((wn >> 5) & 0x3FFFFFFu);
        pos += 3;
        seen_wide |= wide ? 1u : 0u;
        const bool key = f < KF;
        const uint32_t s = !key ? 0u : f == 0 ? s0 : f == 1 ? s1 : s2;
        const uint32_t shift = key ? K * (KF - 1 - f) : 0u;
        const uint32_t qbits = wide ? 53u : 24u;
        const uint32_t wlim = key ? s : qbits;
        const uint32_t pw = words_for(nb, w);
        if ((key && s + K > qbits) || w > wlim || nout > nb ||
            pos + pw + 3 * (uint64_t)nout > len) {
            bad = true;
            break;
        }
        const float eb = u2f(ebt[f]);
        const uint32_t kbits = key ? K : 0u;
        wave_lds_sync();  // previous users of `words` are done
        stage_words<kSteps64>(words, rec + pos, pw, lane);
        wave_lds_sync();
        double y[kItems];
        if (!wide) {
            const float twoeb = 2.0f * eb, lo32 = (float)lo;
            const uint32_t mask = low_mask(w);
#pragma unroll
            for (int j = 0; j < kItems; j++) {
                const uint32_t p = 128 * (j / 2) + 2 * lane + (j & 1);
                const uint32_t v = extract(words, p, w, mask);
                const uint32_t seg = __builtin_amdgcn_ubfe(skey[j / 2], shift + 16u * (j & 1), kbits);
                y[j] = (double)__builtin_fmaf((float)((seg << s) | v), twoeb, lo32);
            }
        } else {
            const double twoeb = 2.0 * (double)eb;
            const uint64_t mask = low_mask64(w);
            const uint32_t mlo = (uint32_t)mask, mhi = (uint32_t)(mask >> 32);
#pragma unroll
            for (int j = 0; j < kItems; j++) {
                const uint32_t p = 128 * (j / 2) + 2 * lane + (j & 1);
                const uint32_t bit = p * w, wd = bit >> 5, sh = bit & 31u;
                const uint32_t a0 = words[wd], a1 = words[wd + 1], a2 = words[wd + 2];
                const uint32_t vlo = __builtin_amdgcn_alignbit(a1, a0, sh) & mlo;
                const uint32_t vhi = __builtin_amdgcn_alignbit(a2, a1, sh) & mhi;
                const uint64_t seg = __builtin_amdgcn_ubfe(skey[j / 2], shift + 16u * (j & 1), kbits);
                const uint64_t q = (seg << s) + (((uint64_t)vhi << 32) | vlo);
                y[j] = __builtin_fma((double)q, twoeb, lo);
            }
        }
        double* yf = reinterpret_cast<double*>(a.y[f].get()) + base;
        if (full && ((reinterpret_cast<uintptr_t>(a.y[f].get()) & 15u) == 0)) {
#pragma unroll
            for (int k = 0; k < kItems / 2; k++) {
                const f64x2 t = {y[2 * k], y[2 * k + 1]};
                __builtin_nontemporal_store(t, reinterpret_cast<f64x2*>(yf + 128 * k + 2 * lane));
            }
        } else {
#pragma unroll
            for (int j = 0; j < kItems; j++) {
                const uint32_t p = 128 * (j / 2) + 2 * lane + (j & 1);
                if (p < nb) yf[p] = y[j];
            }
        }
        pos += pw;
        if (nout) {
            // the outliers overwrite values other lanes stored: the barrier
            // orders those stores first
            __syncthreads();
            const uint32_t* ol = rec + pos;
            bool obad = false;
            for (uint32_t k = lane; k < nout; k += 64) {
                const uint32_t op = ol[3 * k];
                const uint32_t prevp = k ? ol[3 * k - 3] : 0u;
                if (op >= nb || (k && prevp >= op)) obad = true;
                else
                    reinterpret_cast<uint64_t*>(yf)[op] =
                        (uint64_t)ol[3 * k + 1] | ((uint64_t)ol[3 * k + 2] << 32);
            }
            if (__any(obad)) {
                bad = true;
                break;
            }
            pos += 3 * (uint64_t)nout;
        }
    }
    if (bad || pos != len || seen_wide != any_wide) {
        if (lane == 0) *a.err = 1u;
    }
}

__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(5))) void decode_blocks64(DecodeArgs a) {
    __shared__ __align__(16) uint32_t words[kBuf64];
    decode_block64(a, blockIdx.x, words);
    post_header(a);
}

}  // namespace
}  // namespace gpz
