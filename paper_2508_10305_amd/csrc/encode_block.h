// Pieces of the wave-per-block encoders (float32 in encode.hip, float64 in
// encode64.h): quantizer of float32 fields, stable in-block radix sort,
// run-length tables, fixed-length packing, for one block of B = 64 * ITEMS
// particles per wave64.  Lane l owns the ITEMS consecutive particles
// [l*ITEMS, (l+1)*ITEMS) ("blocked"); LDS traffic between the lanes of the
// (one-wave) workgroup is ordered by wave_lds_sync().
#pragma once

#include "gpz_internal.h"

namespace gpz {
namespace {

// The few-blocks form clears for itself what the launches after it count in.
__device__ __forceinline__ void start_few(const EncodeArgs& a, uint32_t b) {
    if (b == 0 && threadIdx.x == 0) {
        *a.wide_flag = 0u;
        *a.done = 0u;
    }
}

constexpr uint32_t kDigitBits = 5;
constexpr uint32_t kDigits = 1u << kDigitBits;
// Digit counters, digit-major: (d, lane) at d*68 + lane (4 pad words per
// digit row, so that the raking scan's 16-byte reads spread over the banks).
// The address is one multiply-add of the digit; the clearing loop writes
// 2304 words (nine 16-byte stores per lane), past the 2176 used.
constexpr uint32_t kRow = 68;
constexpr uint32_t kCounterWords = 64 * 9 * 4;
static_assert(kDigits * kRow <= kCounterWords, "counter rows fit the cleared region");

__device__ __forceinline__ uint32_t counter_addr(uint32_t d, uint32_t lane) {
    return d * kRow + lane;
}

// Padded blocked layout: position p of a block lives at p + 4*(p / ITEMS), so
// lane l's ITEMS consecutive positions start at l*(ITEMS+4) (16-byte aligned,
// spread over the banks).
template <int ITEMS>
__device__ __forceinline__ uint32_t pad_addr(uint32_t p) {
    return p + 4 * (p / ITEMS);
}

// Sort items carry (segment ID << 16) | byte offset of the particle's word
// in the padded blocked layout, so that the per-field permutation reads take
// their LDS address straight from the item.  Once the runs are coded the
// segment IDs are cleared from the items, which leaves the offset alone.
__device__ __forceinline__ uint32_t staged_at(const uint32_t* work, uint32_t offset) {
    return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(work) + offset);
}

// The particle index of an item: padded word p + 4*(p/ITEMS) back to p.
template <int ITEMS>
__device__ __forceinline__ uint32_t index_of(uint32_t item) {
    const uint32_t w = (item & 0xFFFFu) >> 2;
    return w - 4u * (w / (ITEMS + 4));
}

// Quantizer: t = (x - lo) * inv (two IEEE float ops), q = rint(t) when t lies
// in [0, 2^24-1] (else 0); the value stays on the grid only when the float32
// error of xr = fma(q, 2eb, lo) is below eb (which bounds the exact error
// strictly), otherwise it is an outlier stored verbatim.
__device__ __forceinline__ uint32_t quantize(float x, float lo, float inv, float twoeb, float eb,
                                             bool& outlier, bool& in) {
    float t = (x - lo) * inv;
    in = (t >= 0.0f) && (t <= kQMax);
    uint32_t q = in ? (uint32_t)__builtin_rintf(t) : 0u;
    float xr = __builtin_fmaf((float)q, twoeb, lo);
    bool ok = in && (__builtin_fabsf(xr - x) < eb);
    outlier = !ok;
    return q;
}

template <int ITEMS, bool FULL>
__device__ __forceinline__ void load_block(const float* __restrict__ x, uint64_t base, uint32_t nb,
                                           uint32_t lane, float (&v)[ITEMS]) {
    const float* p = x + base + (uint64_t)lane * ITEMS;
    if (FULL && ((reinterpret_cast<uintptr_t>(x) & 15u) == 0)) {
        const f32x4* p4 = reinterpret_cast<const f32x4*>(p);
#pragma unroll
        for (int k = 0; k < ITEMS / 4; k++) {
            f32x4 t = p4[k];  // cached loads: measured faster than non-temporal ones
            v[4 * k + 0] = t.x;
            v[4 * k + 1] = t.y;
            v[4 * k + 2] = t.z;
            v[4 * k + 3] = t.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            uint32_t i = lane * ITEMS + j;
            v[j] = (FULL || i < nb) ? p[j] : 0.0f;
        }
    }
}

// A field of the block after quantization: its minimum lo, the largest code
// over the block's particles, whether no value is an outlier, and whether a
// finite value lies beyond 2^24 - 1 grid steps (the field then needs 64-bit
// steps, Sec. 5.3, which the generic encoder takes).
struct FieldCodes {
    float lo;
    uint32_t qmax;
    bool clean;
    bool wide;
};

// Quantize one field of the block (Sec. 4.1).  Codes are returned as q per
// value for a field without outliers (`clean`), as 2*q + outlier otherwise
// (0 beyond the block).
//
// Fast path, exact for a field without outliers.  Every finite value lies at
// or above the block minimum lo, so t = (x - lo) * inv is never below -0, and
// because no float32 lies strictly between 2^24-1 and 2^24, t <= 2^24-1 holds
// exactly when rint(t) <= 2^24-1.  So a value is on the grid exactly when the
// float32 error of fma(rint(t), 2eb, lo) is below eb and rint(t) does not
// exceed 2^24-1 (a t out of range is NaN, infinite or at least 2^24, and
// fails one of the two).  With q = rint(t) for every value of the field,
// fma(q, 2eb, lo) is the reconstruction the quantizer defines (q = -0 and
// q = +0 give the same result, as lo is never -0).  When any value fails,
// the whole field is quantized again with the quantizer's own steps.
template <int ITEMS, bool FULL>
__device__ __forceinline__ FieldCodes quantize_field(const float (&v)[ITEMS], uint32_t nb,
                                                     uint32_t lane, float inv, float twoeb,
                                                     float eb, uint32_t (&q)[ITEMS]) {
    // Block minimum over the finite values.  +inf is the minimum's identity,
    // so only NaN and -inf have to be skipped: a minimum that propagates NaN
    // over the raw values ends up NaN or -inf in some lane exactly when the
    // block holds one of them, and only then are values filtered one by one.
    // The test is a class test (signalling NaN, quiet NaN, -inf): the
    // compiler lowered the equivalent `m > -inf` under a wave vote to an
    // unordered compare, which a NaN passes.
    float m = __builtin_inff();
#pragma unroll
    for (int j = 0; j < ITEMS; j++)
        m = __builtin_elementwise_minimum(
            m, (FULL || lane * ITEMS + j < nb) ? v[j] : __builtin_inff());
    if (__any(__builtin_amdgcn_classf(m, 7))) {
        m = __builtin_inff();
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            bool ok = (FULL || lane * ITEMS + j < nb) && __builtin_isfinite(v[j]);
            m = fminf(m, ok ? v[j] : __builtin_inff());
        }
    }
    m = wave_min_f32(m);
    const float lo = (m == __builtin_inff() || m == 0.0f) ? 0.0f : m;
    // Every error is below eb exactly when the largest one is.  The maximum
    // propagates NaN (a non-finite value's error), which then fails the test
    // like the value's own comparison would; it takes two errors per
    // instruction where a per-value flag took a compare and a select.
    float emax = 0.0f;
    float rmax = 0.0f;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        const bool valid = FULL || lane * ITEMS + j < nb;
        const float r = __builtin_rintf((v[j] - lo) * inv);
        const float xr = __builtin_fmaf(r, twoeb, lo);
        emax = __builtin_elementwise_maximum(emax, valid ? __builtin_fabsf(xr - v[j]) : 0.0f);
        rmax = fmaxf(rmax, valid ? r : 0.0f);
        q[j] = valid ? (uint32_t)r : 0u;
    }
    uint32_t qmax = wave_max_u32(rmax <= kQMax ? (uint32_t)rmax : 0xFFFFFFFFu);
    if (__all(emax < eb) && qmax <= 0xFFFFFFu) return {lo, qmax, true, false};
    // some value is an outlier: the quantizer's steps, value by value
    uint32_t mx = 0;
    bool far = false;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        const bool valid = FULL || lane * ITEMS + j < nb;
        bool o, in;
        const uint32_t qq = quantize(v[j], lo, inv, twoeb, eb, o, in);
        q[j] = valid ? (qq << 1) | (uint32_t)o : 0u;
        mx = max(mx, valid ? qq : 0u);
        far = far || (valid && !in && __builtin_isfinite(v[j]));
    }
    qmax = wave_max_u32(mx);
    return {lo, qmax, false, __any(far) != 0};
}

// Fixed-length packing (Sec. 4.3): value i of `count` values of width w
// (1 <= w <= 24) goes to bits [i*w, i*w+w) of dst.  Lane l packs its ITEMS
// consecutive values (blocked in v).  Bit positions inside the lane's
// segment, j*w, are the same for every lane, so the lane accumulates into one
// register and flushes on wave-uniform branches; each completed segment word
// is shifted to the lane's start bit with one 64-bit shift and stored into
// LDS staging.  The lane owning bit 0 of a word stores it; a lane whose
// segment starts inside a word ORs its part in after a barrier.  The staged
// words are then copied to dst with coalesced stores.
template <int ITEMS>
__device__ __forceinline__ void pack_generic(const uint32_t (&v)[ITEMS], uint32_t nwords,
                                             uint32_t count, uint32_t w, uint32_t* stage,
                                             uint32_t lane) {
    const bool active = lane * ITEMS < count;
    const uint32_t S = lane * ITEMS * w;            // first bit of the lane's segment
    const uint32_t w0 = S >> 5, shl = S & 31u;
    const uint32_t lastw = (S + ITEMS * w - 1) >> 5;  // last word the segment touches
    uint32_t acc = 0u, prev = 0u, first = 0u;
    uint32_t k = 0, pos = 0;  // segment word index and bit position in it (uniform)
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        acc |= v[j] << pos;
        pos += w;
        if (pos >= 32u) {
            const uint32_t gi = w0 + k;
            const uint32_t word = (uint32_t)((((uint64_t)acc << 32) | prev) >> (32u - shl));
            if (active && gi < nwords && (k > 0 || shl == 0)) stage[gi] = word;
            if (k == 0) first = acc;
            prev = acc;
            pos -= 32u;
            acc = pos ? v[j] >> (w - pos) : 0u;
            k++;
        }
    }
    if (pos > 0u) {  // last, partly filled segment word
        const uint32_t gi = w0 + k;
        const uint32_t word = (uint32_t)((((uint64_t)acc << 32) | prev) >> (32u - shl));
        if (active && gi < nwords && (k > 0 || shl == 0)) stage[gi] = word;
        if (k == 0) first = acc;
        prev = acc;
        k++;
    }
    if (shl != 0u) {  // spill-over of the segment's top bits into one more word
        const uint32_t gi = w0 + k;
        if (active && gi <= lastw && gi < nwords) stage[gi] = prev >> (32u - shl);
    }
    wave_lds_sync();
    if (active && shl != 0u && w0 < nwords) atomicOr(&stage[w0], first << shl);
}

// The same packing for 16 values per lane at a width W known at compile
// time: every shift is a constant and no branch depends on the bit position.
// Lane l's values take bits [16*W*l, 16*W*(l+1)) of the array.  For even W
// that is W/2 whole words.  For odd W the lanes of a pair 2m, 2m+1 share one
// word (the even lane's last, the odd lane's first): the even lane completes
// it with the odd lane's low 16 bits, moved over by a DPP lane shift within
// the row, and stores it.  Every lane packs (values past the array's count
// are zero), and words past the array's end land in the staging buffer
// without being copied out.
// `dst` is the lane's first word in the staging buffer, stage + lane*W/2
// (rounded down), computed by the caller from the run-time width so that the
// compiler has no per-width address to keep live across the field loop.
template <int W>
__device__ __forceinline__ void pack16(const uint32_t (&v)[16], uint32_t* dst, uint32_t lane) {
    constexpr int NS = (16 * W + 31) / 32;  // words of the segment, from its first bit
    uint32_t s[NS];
#pragma unroll
    for (int k = 0; k < NS; k++) s[k] = 0u;
#pragma unroll
    for (int j = 0; j < 16; j++) {
        const int bit = j * W, k = bit >> 5, sh = bit & 31;
        s[k] |= v[j] << sh;
        if (sh + W > 32) s[k + 1] |= v[j] >> (32 - sh);
    }
    if constexpr (W % 2 == 0) {
#pragma unroll
        for (int k = 0; k < W / 2; k++) dst[k] = s[k];
    } else {
        constexpr int H = (W - 1) / 2;  // whole words of an even lane before the shared one
        const bool odd = (lane & 1u) != 0u;
        const uint32_t nxt = dpp<kRowShl1>(s[0] << 16);
#pragma unroll
        for (int t = 0; t <= H; t++) {
            const uint32_t ev = t < H ? s[t] : (s[H] | nxt);
            const uint32_t od = t ? __builtin_amdgcn_alignbit(s[t], s[t - 1], 16) : 0u;
            if (t > 0 || !odd) dst[t] = odd ? od : ev;
        }
    }
}

#define GPZ_PACK16_CASE(W) \
    case W: pack16<W>(v, first, lane); break;

// Fixed-length packing of one array (Sec. 4.3) into the LDS staging buffer:
// value i of `count` values of width w goes to bits [i*w, i*w+w) of it.
template <int ITEMS>
__device__ __forceinline__ void pack_stage(const uint32_t (&v)[ITEMS], uint32_t count, uint32_t w,
                                           uint32_t* stage, uint32_t lane) {
    const uint32_t nwords = words_for(count, w);
    if (nwords == 0) return;
    if constexpr (ITEMS == 16) {
        uint32_t* first = stage + ((lane * w) >> 1);
        switch (w) {
            GPZ_PACK16_CASE(1) GPZ_PACK16_CASE(2) GPZ_PACK16_CASE(3) GPZ_PACK16_CASE(4)
            GPZ_PACK16_CASE(5) GPZ_PACK16_CASE(6) GPZ_PACK16_CASE(7) GPZ_PACK16_CASE(8)
            GPZ_PACK16_CASE(9) GPZ_PACK16_CASE(10) GPZ_PACK16_CASE(11) GPZ_PACK16_CASE(12)
            GPZ_PACK16_CASE(13) GPZ_PACK16_CASE(14) GPZ_PACK16_CASE(15) GPZ_PACK16_CASE(16)
            GPZ_PACK16_CASE(17) GPZ_PACK16_CASE(18) GPZ_PACK16_CASE(19) GPZ_PACK16_CASE(20)
            GPZ_PACK16_CASE(21) GPZ_PACK16_CASE(22) GPZ_PACK16_CASE(23) GPZ_PACK16_CASE(24)
            default: pack_generic<ITEMS>(v, nwords, count, w, stage, lane); break;
        }
    } else {
        pack_generic<ITEMS>(v, nwords, count, w, stage, lane);
    }
}

// The nwords staged words to dst with coalesced stores, four words per lane
// at a time: the four staging reads are all issued before the stores, so
// they cost one LDS round trip, not four.  Whole 256-word steps store
// unconditionally, at 32-bit byte offsets from the array's scalar base; only
// the last, partial step is predicated.  Reads past nwords stay inside the
// staging buffer (its size is checked against the largest array, B values
// of 24 bits) and are never stored.
template <int ITEMS>
__device__ __forceinline__ void copy_out(uint32_t nwords, uint32_t* __restrict__ dst,
                                         const uint32_t* stage, uint32_t lane) {
    uint8_t* const base = reinterpret_cast<uint8_t*>(dst);
    const uint32_t whole = nwords & ~255u;
    for (uint32_t i0 = 0; i0 < whole; i0 += 256) {
        uint32_t t[4];
#pragma unroll
        for (int u = 0; u < 4; u++) t[u] = stage[i0 + 64 * u + lane];
#pragma unroll
        for (int u = 0; u < 4; u++)
            *reinterpret_cast<uint32_t*>(base + 4u * (i0 + 64u * u + lane)) = t[u];
    }
    if (whole < nwords) {
        uint32_t t[4];
#pragma unroll
        for (int u = 0; u < 4; u++) t[u] = stage[whole + 64 * u + lane];
        // keeps the compiler from sinking a read into its store's branch
        asm volatile("" : : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]));
#pragma unroll
        for (int u = 0; u < 4; u++)
            if (whole + 64 * u + lane < nwords)
                *reinterpret_cast<uint32_t*>(base + 4u * (whole + 64u * u + lane)) = t[u];
    }
}

// Fixed-length packing of one array into dst (Sec. 4.3), staged in LDS and
// copied out with coalesced stores.
template <int ITEMS>
__device__ __forceinline__ void pack_array(const uint32_t (&v)[ITEMS], uint32_t count, uint32_t w,
                                           uint32_t* __restrict__ dst, uint32_t* stage,
                                           uint32_t lane) {
    const uint32_t nwords = words_for(count, w);
    if (nwords == 0) return;
    pack_stage<ITEMS>(v, count, w, stage, lane);
    wave_lds_sync();
    copy_out<ITEMS>(nwords, dst, stage, lane);
    wave_lds_sync();
}

// One stable LSD pass over 5 key bits starting at bit `sh` of the key
// (key = kv >> 16).  Each lane counts its own items per digit (LDS atomics on
// its private counter column give the within-lane rank), a raking scan in
// (digit, lane) order gives every (digit, lane) its first slot, and items are
// scattered to their slots and read back blocked.
template <int ITEMS, bool FULL, bool LEAN = false>
__device__ __forceinline__ void radix_pass(uint32_t (&kv)[ITEMS], uint32_t sh, uint32_t nb,
                                           uint32_t lane, uint32_t* cnt, uint32_t* kvbuf) {
    uint4* c4 = reinterpret_cast<uint4*>(cnt);
#pragma unroll
    for (int k = 0; k < 9; k++) c4[lane * 9 + k] = make_uint4(0, 0, 0, 0);
    wave_lds_sync();
    uint32_t rank[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        const uint32_t d = __builtin_amdgcn_ubfe(kv[j], 16 + sh, kDigitBits);
        if (FULL || lane * ITEMS + j < nb) rank[j] = atomicAdd(&cnt[counter_addr(d, lane)], 1u);
        else rank[j] = 0u;
    }
    wave_lds_sync();
    if constexpr (LEAN) {
        // as below, in two halves of 16 counters (the counters are read
        // twice), and the digits extracted again after the scan: fewer
        // registers held across it
        uint4* row = reinterpret_cast<uint4*>(cnt + (lane >> 1) * kRow + (lane & 1) * 32);
        uint32_t run = 0;
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const uint4 t = row[k];
            run += t.x + t.y + t.z + t.w;
        }
        uint32_t before = wave_incl_scan_u32(run) - run;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            uint32_t c[16];
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const uint4 t = row[4 * h + k];
                c[4 * k + 0] = t.x;
                c[4 * k + 1] = t.y;
                c[4 * k + 2] = t.z;
                c[4 * k + 3] = t.w;
            }
#pragma unroll
            for (int k = 0; k < 16; k++) {
                const uint32_t t = c[k];
                c[k] = before;
                before += t;
            }
#pragma unroll
            for (int k = 0; k < 4; k++)
                row[4 * h + k] = make_uint4(c[4 * k], c[4 * k + 1], c[4 * k + 2], c[4 * k + 3]);
            wave_lds_sync();
        }
#pragma unroll
        for (int j = 0; j < ITEMS; j++) asm volatile("" : "+v"(kv[j]));
    } else {
        // lane r scans flat entries [32r, 32r+32) of (digit, lane) order:
        // digit r/2, lanes 32*(r%2) .. 32*(r%2)+31, contiguous in its row
        uint4* row = reinterpret_cast<uint4*>(cnt + (lane >> 1) * kRow + (lane & 1) * 32);
        uint32_t c[32];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            uint4 t = row[k];
            c[4 * k + 0] = t.x;
            c[4 * k + 1] = t.y;
            c[4 * k + 2] = t.z;
            c[4 * k + 3] = t.w;
        }
        uint32_t run = 0;
#pragma unroll
        for (int k = 0; k < 32; k++) {
            uint32_t t = c[k];
            c[k] = run;
            run += t;
        }
        uint32_t before = wave_incl_scan_u32(run) - run;
#pragma unroll
        for (int k = 0; k < 8; k++)
            row[k] = make_uint4(c[4 * k] + before, c[4 * k + 1] + before, c[4 * k + 2] + before,
                                c[4 * k + 3] + before);
    }
    wave_lds_sync();
    // All counter reads are issued before the first scatter store: a store
    // between them would make every read wait for the one before it.
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        const uint32_t d = __builtin_amdgcn_ubfe(kv[j], 16 + sh, kDigitBits);
        rank[j] += cnt[counter_addr(d, lane)];
    }
#pragma unroll
    for (int j = 0; j < ITEMS; j++)
        if (FULL || lane * ITEMS + j < nb) kvbuf[pad_addr<ITEMS>(rank[j])] = kv[j];
    wave_lds_sync();
    const uint4* mine = reinterpret_cast<const uint4*>(kvbuf + lane * (ITEMS + 4));
#pragma unroll
    for (int k = 0; k < ITEMS / 4; k++) {
        uint4 t = mine[k];
        kv[4 * k + 0] = t.x;
        kv[4 * k + 1] = t.y;
        kv[4 * k + 2] = t.z;
        kv[4 * k + 3] = t.w;
    }
    wave_lds_sync();
}

// A field's codes (q, or 2*q + outlier for a field with outliers) into lane
// l's LDS row.  A key field also needs the largest of its in-segment offsets
// (the low `width` bits of q); a field with outliers needs their number.
template <int ITEMS, bool KEY>
__device__ __forceinline__ void stage_codes(const uint32_t (&q)[ITEMS], uint32_t width, bool clean,
                                            uint4* mine, uint32_t& vmax, uint32_t& no) {
    if (KEY) {
#pragma unroll
        for (int j = 0; j < ITEMS; j++)
            vmax = max(vmax, __builtin_amdgcn_ubfe(q[j], clean ? 0u : 1u, width));
    }
    if (!clean) {
#pragma unroll
        for (int j = 0; j < ITEMS; j++) no += q[j] & 1u;
    }
#pragma unroll
    for (int k = 0; k < ITEMS / 4; k++)
        mine[k] = make_uint4(q[4 * k], q[4 * k + 1], q[4 * k + 2], q[4 * k + 3]);
}

// Runs of the sorted segment IDs (Sec. 4.3): uniq[k] is the k-th distinct ID
// and start[k] the sorted position where its run begins, k < U, with
// start[U] = nb.  Lane l takes runs l*ITEMS .. l*ITEMS+ITEMS-1 (0 beyond U).
// Each lane reads its ITEMS words with 16-byte loads, unconditionally (the
// buffers hold B words, entries from U on are ignored), so no read waits for
// another.  Runs past U are cleared with a per-lane bit mask: a compare per
// run would give the compiler U-dependent lane masks to keep (and spill)
// across the whole field loop, so U is also made opaque here.
template <int ITEMS>
__device__ __forceinline__ void load_runs(const uint32_t* src, uint32_t lane,
                                          uint32_t (&r)[ITEMS]) {
    const uint4* p = reinterpret_cast<const uint4*>(src + lane * ITEMS);
#pragma unroll
    for (int k = 0; k < ITEMS / 4; k++) {
        uint4 t = p[k];
        r[4 * k + 0] = t.x;
        r[4 * k + 1] = t.y;
        r[4 * k + 2] = t.z;
        r[4 * k + 3] = t.w;
    }
}

// Bit j set when run lane*ITEMS + j exists (j < ITEMS <= 32).
template <int ITEMS>
__device__ __forceinline__ uint32_t run_mask(uint32_t U, uint32_t lane) {
    asm volatile("" : "+s"(U));
    const int c = min(max((int)U - (int)(lane * ITEMS), 0), ITEMS);
    return c >= 32 ? ~0u : (1u << c) - 1u;
}

// ID gaps minus one; the first ID counts from -1, so its gap is the ID.
template <int ITEMS>
__device__ __forceinline__ void run_gaps(const uint32_t* uniq, uint32_t U, uint32_t lane,
                                         uint32_t (&v)[ITEMS]) {
    uint32_t r[ITEMS];
    load_runs<ITEMS>(uniq, lane, r);
    const uint32_t m = run_mask<ITEMS>(U, lane);
    uint32_t before = (uint32_t)__shfl_up((int)r[ITEMS - 1], 1);
    if (lane == 0) before = 0xFFFFFFFFu;
#pragma unroll
    for (int j = 0; j < ITEMS; j++)
        v[j] = (r[j] - (j ? r[j - 1] : before) - 1u) & (uint32_t)__builtin_amdgcn_sbfe(m, j, 1);
}

// Run lengths minus one: start[i+1] - start[i] - 1 (start[U] = nb).
template <int ITEMS>
__device__ __forceinline__ void run_counts(const uint32_t* start, uint32_t U, uint32_t lane,
                                           uint32_t (&v)[ITEMS]) {
    uint32_t r[ITEMS];
    load_runs<ITEMS>(start, lane, r);
    const uint32_t after = start[lane * ITEMS + ITEMS];
    const uint32_t m = run_mask<ITEMS>(U, lane);
#pragma unroll
    for (int j = 0; j < ITEMS; j++)
        v[j] = ((j + 1 < ITEMS ? r[j + 1] : after) - r[j] - 1u) &
               (uint32_t)__builtin_amdgcn_sbfe(m, j, 1);
}

// Run-length coding (Sec. 4.3) of the sorted items kv (segment ID << 16 | LDS
// offset): the distinct IDs go to uniq[0, U), the positions their runs begin
// at to start[0, U], start[U] = nb.  Returns U; the IDs are cleared from the
// items, which are only LDS offsets (the permutation) from here on.  `start`
// follows `uniq` by B words, both followed by the lanes' scratch words.
template <int ITEMS, bool FULL>
__device__ __forceinline__ uint32_t code_runs(uint32_t (&kv)[ITEMS], uint32_t nb, uint32_t lane,
                                              uint32_t* uniq, uint32_t* start) {
    constexpr uint32_t B = 64 * ITEMS;
    const uint32_t prev = (uint32_t)__shfl_up((int)(kv[ITEMS - 1] >> 16), 1);
    uint32_t nflag = 0;
    bool flag[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        uint32_t p = lane * ITEMS + j;
        uint32_t key = kv[j] >> 16;
        uint32_t before = j == 0 ? prev : (kv[j - 1] >> 16);
        flag[j] = (FULL || p < nb) && (p == 0 || key != before);
        nflag += flag[j];
    }
    uint32_t incl = wave_incl_scan_u32(nflag);
    const uint32_t U = readlane(incl, 63);
    // Every item stores, without branches: a run start at its rank k, any
    // other item to a scratch word of its lane past the tables.
    uint32_t k = incl - nflag;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        uniq[flag[j] ? k : 2 * B + 64 + lane] = kv[j] >> 16;
        start[flag[j] ? k : B + 128 + lane] = lane * ITEMS + j;
        k += flag[j] ? 1u : 0u;
    }
    if (lane == 0) start[U] = nb;
    wave_lds_sync();
#pragma unroll
    for (int j = 0; j < ITEMS; j++) kv[j] &= 0xFFFFu;
    return U;
}

}  // namespace
}  // namespace gpz
