// Block encoder: GPZ stages 1-3 (Sec. 4.1 quantization, Sec. 4.2 in-block
// sort, Sec. 4.3 run-length / delta / fixed-length coding) for one block of
// B particles per wave64, writing the block's record into its workspace slot
// and its length (first step of the Sec. 4.4 compaction; the scan and copy
// kernels finish it).  An alternative single-pass compaction is also built:
// the block publishes its length, finds its offset in the stream by a
// decoupled look-back over the lengths of the blocks before it, and copies
// its record there itself.
//
// Lane layout: lane l owns the ITEMS = B/64 consecutive particles
// [l*ITEMS, (l+1)*ITEMS) of its block ("blocked"), so per-lane sequential
// order followed by lane order is input order; that is what makes the LDS
// radix sort stable.  One wave per workgroup: LDS traffic between lanes is
// ordered by wave_lds_sync(), which waits for nothing (a wave's LDS
// operations execute in issue order); __syncthreads() remains only where
// global-memory stores of the block must be ordered.  Full blocks take a path
// without per-item bounds checks; only the last block of a snapshot can be
// partial.
#include "encode64.h"
#include "encode_block.h"
#include "place.h"

namespace gpz {
namespace {

// ------------------------------------------------------------ compaction
// Look-back word of a block: (value << 2) | flag, flag 1 = the block's own
// record length is known, 2 = the inclusive prefix (words of all records up
// to and including this block) is known, 0 = nothing yet.
constexpr uint64_t kFlagLen = 1u, kFlagIncl = 2u;

__device__ __forceinline__ uint64_t load_state(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_state(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Exclusive prefix (in words) of the record lengths of blocks 0..b-1.  Every
// block with a smaller index was started before this one (tickets), so the
// waits below always end.  Lane i inspects block top - i; the
// window moves back 64 blocks at a time until it meets an inclusive prefix.
__device__ __forceinline__ uint64_t exclusive_offset(uint64_t* state, uint32_t b, uint32_t len,
                                                     uint32_t lane) {
    if (lane == 0) store_state(state + b, ((uint64_t)len << 2) | (b == 0 ? kFlagIncl : kFlagLen));
    if (b == 0) return 0;
    uint64_t excl = 0;
    int64_t top = (int64_t)b - 1;
    for (;;) {
        const int64_t p = top - (int64_t)lane;
        const uint64_t st = p >= 0 ? load_state(state + p) : kFlagIncl;
        const uint64_t flag = st & 3u;
        const uint64_t incl = __ballot(flag == kFlagIncl);
        const uint64_t pending = __ballot(flag == 0);
        // lanes up to and including the nearest inclusive prefix
        const uint64_t upto = incl ? ((incl & (~incl + 1)) << 1) - 1 : ~0ull;
        if (pending & upto) {
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        excl += wave_sum_u64(((upto >> lane) & 1u) ? (st >> 2) : 0u);
        if (incl) break;
        top -= 64;
    }
    if (lane == 0) store_state(state + b, ((excl + len) << 2) | kFlagIncl);
    return excl;
}

// Stream header and error-bound table (format v1).
__device__ __forceinline__ void write_header(const EncodeArgs& a, uint32_t lane) {
    uint32_t* out = a.out;
    if (lane == 0) {
        out[0] = kMagic;
        out[1] = kVersion;
        out[2] = (uint32_t)(a.n & 0xFFFFFFFFu);
        out[3] = (uint32_t)(a.n >> 32);
        out[4] = a.F;
        out[5] = a.B;
        out[6] = a.K | (a.KF << 8);
        out[7] = a.nblocks;
    }
    uint32_t* ebt = out + kHeaderWords + 2 * nsuper_of(a.nblocks);
    for (uint32_t f = lane; f < a.F; f += 64) ebt[f] = f2u(a.eb[f]);
}

__device__ __forceinline__ void publish_size(const EncodeArgs& a, uint64_t total, uint32_t lane) {
    if (lane == 0) {
        *a.total_bytes = total;
        if (a.ext_bytes) *a.ext_bytes = total;
    }
    if (total <= a.capacity) write_header(a, lane);
}

// Block b's record (len words at rec) goes to its final offset; the block
// also writes its length-table entry, the superblock entry when it opens a
// superblock, and, as the last block, the stream size and header.  Nothing
// is written past the output capacity.
__device__ __forceinline__ void place_record(const EncodeArgs& a, uint32_t b, const uint32_t* rec,
                                             uint32_t len, uint32_t lane) {
    __syncthreads();  // the record's stores by all lanes before they are read back
    const uint64_t excl = exclusive_offset(a.state, b, len, lane);
    const uint64_t capw = a.capacity / 4;
    const uint64_t sup_at = kHeaderWords;
    const uint64_t lt_at = kHeaderWords + 2 * nsuper_of(a.nblocks) + a.F;
    uint32_t* out = a.out;
    if (lane == 0) {
        if (lt_at + b < capw) out[lt_at + b] = len;
        if (b % kSuper == 0) {
            const uint64_t at = sup_at + 2 * (b / kSuper);
            if (at + 1 < capw) {
                out[at] = (uint32_t)(excl & 0xFFFFFFFFu);
                out[at + 1] = (uint32_t)(excl >> 32);
            }
        }
    }
    const uint64_t off = a.prefix + excl;
    if (off + len <= capw) {
        uint32_t* dst = out + off;
        for (uint32_t k = lane; k < len; k += 256) {
            uint32_t v[4];
#pragma unroll
            for (int i = 0; i < 4; i++) v[i] = k + 64 * i < len ? rec[k + 64 * i] : 0u;
#pragma unroll
            for (int i = 0; i < 4; i++)
                if (k + 64 * i < len) dst[k + 64 * i] = v[i];
        }
    }
    if (b == a.nblocks - 1) publish_size(a, 4 * (off + len), lane);
}

// The block's LDS: one region whose phases reuse it.
//  - sort: radix counters (kCounterWords, 68-word digit rows) and, aliased
//    with them, the scatter target in the padded blocked layout (64*(ITEMS+4)
//    words): each pass reads every counter it needs before its first
//    scatter store, and a wave's LDS operations execute in issue order;
//  - run tables: uniq[0, B), start[0, B] at B, per-lane scratch words for
//    the branch-free run stores at 2B + 64 and 2B + 128;
//  - field loop: the field's codes in the padded blocked layout at 0, and
//    the packer's staging from kStageAt (read in steps of 256 words; the
//    widest array, B values of 24 bits, stays inside).
template <int ITEMS>
struct EncodeSmem {
    static constexpr uint32_t B = 64 * ITEMS;
    static constexpr uint32_t kStageAt = 64 * (ITEMS + 4);
    static constexpr uint32_t kStageWords = (48 * ITEMS + 255) / 256 * 256;
    static constexpr uint32_t kA = kCounterWords > 2 * B + 192 ? kCounterWords : 2 * B + 192;
    static constexpr uint32_t kWords =
        kA > kStageAt + kStageWords ? kA : kStageAt + kStageWords;
    static_assert(64 * (ITEMS + 4) <= kWords, "scatter target inside the region");
    __align__(16) uint32_t buf[kWords];
};

// EARLY: how many fields after the key fields are loaded and quantized with
// them, before the sort (at most three); the others are loaded and quantized
// in the field loop.  With none, fewer values are held across the sort.
template <int ITEMS, bool FULL, bool SINGLE, int EARLY = 3, int FORM = kPlain>
__device__ __forceinline__ void encode_block(const EncodeArgs& a, uint32_t b, uint32_t nb,
                                             uint32_t* work) {
    uint32_t* const stage = work + EncodeSmem<ITEMS>::kStageAt;
    constexpr uint32_t B = 64 * ITEMS;
    const uint32_t lane = threadIdx.x;
    const uint64_t base = (uint64_t)b * B;
    const uint32_t F = a.F, K = a.K, KF = a.KF;
    uint32_t* __restrict__ rec = a.temp + (uint64_t)b * a.slot_words;
    const uint32_t cap = 1 + F * nb;  // raw record length

    // ---- Stage 1 (Sec. 4.1): key axes -- block minimum, grid index, segment shift
    // The loads of the key fields and of up to three other fields are all
    // issued here, before any store of the block: vector memory operations
    // complete in issue order, so a load issued behind the record's stores
    // would wait for them.
    float xk[3][ITEMS], xo[3][ITEMS];
#pragma unroll
    for (int ax = 0; ax < 3; ax++)
        if ((uint32_t)ax < KF) load_block<ITEMS, FULL>(a.x[ax], base, nb, lane, xk[ax]);
#pragma unroll
    for (int e = 0; e < EARLY; e++)
        if (KF + e < F) load_block<ITEMS, FULL>(a.x[KF + e], base, nb, lane, xo[e]);
    // codes are 2*q + outlier (Sec. 4.1)
    uint32_t qk[3][ITEMS];
    FieldCodes ck[3];
    uint32_t sk[3];
#pragma unroll
    for (int ax = 0; ax < 3; ax++) {
        sk[ax] = 0;
        ck[ax] = {0.0f, 0u, true};
        if ((uint32_t)ax < KF) {
            ck[ax] = quantize_field<ITEMS, FULL>(xk[ax], nb, lane, a.inv[ax], a.twoeb[ax],
                                                 a.eb[ax], qk[ax]);
            const uint32_t W = bit_width(ck[ax].qmax);
            sk[ax] = W > K ? W - K : 0;
        } else {
#pragma unroll
            for (int j = 0; j < ITEMS; j++) qk[ax][j] = 0;
        }
    }
    // the other early fields
    uint32_t qo[3][ITEMS];
    FieldCodes co[3];
#pragma unroll
    for (int e = 0; e < 3; e++) {
        co[e] = {0.0f, 0u, true};
        if (e < EARLY && KF + e < F) {
            const uint32_t f = KF + e;
            co[e] = quantize_field<ITEMS, FULL>(xo[e], nb, lane, a.inv[f], a.twoeb[f], a.eb[f],
                                                qo[e]);
        } else {
#pragma unroll
            for (int j = 0; j < ITEMS; j++) qo[e][j] = 0;
        }
    }

    // A field whose grid needs more than 24 bits: the generic encoder codes
    // the block (three-step compaction); the single pass, which cannot wait
    // for it, stores the block raw.
    bool wide = ck[0].wide || ck[1].wide || ck[2].wide || co[0].wide || co[1].wide || co[2].wide;
    if (!SINGLE && wide) {
        defer_block<FORM>(a, b, lane);
        return;
    }

    // Linearised segment ID (axis 0 most significant), packed with the index.
    uint32_t kv[ITEMS];
    uint32_t keyor = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        uint32_t key = 0;
#pragma unroll
        for (int ax = 0; ax < 3; ax++)
            if ((uint32_t)ax < KF)
                key = (key << K) | (qk[ax][j] >> (sk[ax] + (ck[ax].clean ? 0u : 1u)));
        uint32_t i = lane * ITEMS + j;
        kv[j] = (key << 16) | (4u * pad_addr<ITEMS>(i));
        if (FULL || i < nb) keyor |= key;
    }
    keyor = wave_or_u32(keyor);

    // ---- Stage 2 (Sec. 4.2): stable in-block sort by segment ID
    const uint32_t keybits = K * KF;
    for (uint32_t sh = 0; sh < keybits; sh += kDigitBits) {
        if (((keyor >> sh) & (kDigits - 1)) == 0) continue;  // identity pass
        radix_pass<ITEMS, FULL, EARLY == 0>(kv, sh, nb, lane, work, work);
    }

    // ---- Stage 3 (Sec. 4.3): run-length coding of the sorted IDs
    uint32_t* uniq = work;
    uint32_t* start = work + B;
    const uint32_t U = code_runs<ITEMS, FULL>(kv, nb, lane, uniq, start);
    // delta coding of the distinct IDs (stored as delta - 1) and counts - 1,
    // kept in registers until they are packed
    uint32_t gv[ITEMS], cv[ITEMS];
    run_gaps<ITEMS>(uniq, U, lane, gv);
    run_counts<ITEMS>(start, U, lane, cv);
    uint32_t gmax = 0, cmax = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        gmax = max(gmax, gv[j]);
        cmax = max(cmax, cv[j]);
    }
    const uint32_t w_gap = bit_width(wave_max_u32(gmax));
    const uint32_t w_cnt = bit_width(wave_max_u32(cmax));
    if (lane == 0) {
        rec[0] = U << 2;
        rec[1] = w_gap | (w_cnt << 5) | (sk[0] << 10) | (sk[1] << 15) | (sk[2] << 20);
    }

    // ---- arrays in record order: gaps, counts, then one section per field
    uint32_t pos = 2;
    bool over = wide;  // (single pass only: such a block is stored raw)
    const uint32_t gw = words_for(U, w_gap), cw = words_for(U, w_cnt);
    // Each array's packed words leave the staging buffer while the next
    // field's permutation reads are in flight (one LDS round trip for both):
    // `pend` words staged for `pend_dst` are still to be copied out.
    uint32_t pend = 0;
    uint32_t* pend_dst = rec;
    if (pos + gw + cw > cap) {
        over = true;
    } else {
        wave_lds_sync();  // uniq/start reads done before `work` is reused
        pack_array<ITEMS>(gv, U, w_gap, rec + pos, stage, lane);
        pack_stage<ITEMS>(cv, U, w_cnt, stage, lane);
        pend = cw;
        pend_dst = rec + pos + gw;
        pos += gw + cw;
    }
    // One field's section once its codes are staged in LDS (input order, at
    // `work` in the padded blocked layout): lo and field word, the codes
    // permuted to sorted order (a key field's in-segment offsets: its low
    // `width` bits), packed; its outliers.  Returns false when the block is
    // stored raw (or, for a wide field, left to the generic encoder).
    auto section = [&](uint32_t f, const FieldCodes& c, bool key, uint32_t width, uint32_t vmax,
                       uint32_t no) -> bool {
        if (wide) {
            over = true;
            return false;
        }
        const uint32_t w = bit_width(key ? wave_max_u32(vmax) : c.qmax);
        const uint32_t nout = c.clean ? 0u : wave_sum_u32(no);
        if (pos + 2 + words_for(nb, w) + 2 * nout > cap) {
            over = true;
            return false;
        }
        if (lane == 0) {
            rec[pos] = f2u(c.lo);
            rec[pos + 1] = w | (nout << 5);
        }
        pos += 2;
        // permute to sorted order through LDS
        wave_lds_sync();
        // the packed value: q of a clean non-key field as it is, else the
        // code's grid index (without the outlier bit) cut to `width` bits
        uint32_t vals[ITEMS];
        if (!key && c.clean) {
#pragma unroll
            for (int j = 0; j < ITEMS; j++)
                vals[j] = (FULL || lane * ITEMS + j < nb) ? staged_at(work, kv[j]) : 0u;
        } else {
            const uint32_t s0 = c.clean ? 0u : 1u;
#pragma unroll
            for (int j = 0; j < ITEMS; j++)
                vals[j] = (FULL || lane * ITEMS + j < nb)
                              ? __builtin_amdgcn_ubfe(staged_at(work, kv[j]), s0, width)
                              : 0u;
        }
        if (pend) {
            wave_lds_sync();
            copy_out<ITEMS>(pend, pend_dst, stage, lane);
        }
        wave_lds_sync();  // the staged words are read before they are replaced
        pack_stage<ITEMS>(vals, nb, w, stage, lane);
        pend = words_for(nb, w);
        pend_dst = rec + pos;
        pos += pend;
        if (nout) {
            // outlier flags of the sorted positions, read again from the staging
            uint32_t flags = 0;
#pragma unroll
            for (int j = 0; j < ITEMS; j++)
                if ((FULL || lane * ITEMS + j < nb) &&
                    (staged_at(work, kv[j]) & 1u))
                    flags |= 1u << j;
            const uint32_t cnt = __builtin_popcount(flags);
            uint32_t k = wave_incl_scan_u32(cnt) - cnt;
            uint32_t* ol = rec + pos;
            const float* xf = a.x[f] + base;
#pragma unroll
            for (int j = 0; j < ITEMS; j++) {
                if ((flags >> j) & 1u) {
                    ol[2 * k] = lane * ITEMS + j;
                    ol[2 * k + 1] = f2u(xf[index_of<ITEMS>(kv[j])]);
                    k++;
                }
            }
            pos += 2 * nout;
        }
        wave_lds_sync();  // staging reads done before the next field overwrites it
        return true;
    };
    uint4* const mine = reinterpret_cast<uint4*>(work + lane * (ITEMS + 4));
    if constexpr (EARLY == 0) {
        // The key fields' codes are in registers; each other field is
        // fetched while its predecessor is staged and packed.
        for (uint32_t f = 0; f < KF && !over; f++) {
            // the permutation's LDS offsets are recomputed per field instead
            // of being held in registers across the loop
#pragma unroll
            for (int j = 0; j < ITEMS; j++) asm volatile("" : "+v"(kv[j]));
            FieldCodes c{0.0f, 0u, true, false};
            uint32_t width = 0, vmax = 0, no = 0;
            // one wave-uniform branch per source, each reading its own
            // registers (the empty asm keeps the compiler from merging the
            // branches into a select per value)
            switch (f) {
#define GPZ_STAGE(N)                                                        \
    case N:                                                                 \
        c = ck[N];                                                          \
        width = sk[N];                                                      \
        stage_codes<ITEMS, true>(qk[N], width, c.clean, mine, vmax, no);    \
        asm volatile("");                                                   \
        break;
                GPZ_STAGE(0) GPZ_STAGE(1) GPZ_STAGE(2)
#undef GPZ_STAGE
            }
            if (!section(f, c, true, width, vmax, no)) break;
        }
        float xn[ITEMS];
        if (KF < F && !over) load_block<ITEMS, FULL>(a.x[KF], base, nb, lane, xn);
        for (uint32_t f = KF; f < F && !over; f++) {
#pragma unroll
            for (int j = 0; j < ITEMS; j++) asm volatile("" : "+v"(kv[j]));
            uint32_t q[ITEMS];
            const FieldCodes c =
                quantize_field<ITEMS, FULL>(xn, nb, lane, a.inv[f], a.twoeb[f], a.eb[f], q);
            if (f + 1 < F) load_block<ITEMS, FULL>(a.x[f + 1], base, nb, lane, xn);
            wide = wide || c.wide;
            uint32_t vmax = 0, no = 0;
            stage_codes<ITEMS, false>(q, 24u, c.clean, mine, vmax, no);
            if (!section(f, c, false, 24u, vmax, no)) break;
        }
    } else {
        for (uint32_t f = 0; f < F && !over; f++) {
            FieldCodes c{0.0f, 0u, true, false};
            uint32_t width = 24, vmax = 0, no = 0;
            bool key = false;
            // The field's codes go to LDS in input order (for the
            // permutation).  Key fields and the early fields are already in
            // registers: one wave-uniform branch per source, each reading
            // its own registers (the empty asm keeps the compiler from
            // merging the branches into a select per value).  Later fields
            // are loaded and quantized here.  The packed value is the code's
            // in-segment offset for a key field (its low sk bits), the whole
            // code otherwise.
            const uint32_t src = f < KF ? f : 3 + (f - KF);
            switch (src) {
#define GPZ_STAGE(N, QA, C, KEY, WIDTH)                                  \
    case N:                                                              \
        c = C;                                                           \
        key = KEY;                                                       \
        width = WIDTH;                                                   \
        stage_codes<ITEMS, KEY>(QA, width, c.clean, mine, vmax, no);     \
        asm volatile("");                                                \
        break;
                GPZ_STAGE(0, qk[0], ck[0], true, sk[0])
                GPZ_STAGE(1, qk[1], ck[1], true, sk[1])
                GPZ_STAGE(2, qk[2], ck[2], true, sk[2])
                GPZ_STAGE(3, qo[0], co[0], false, 24u)
                GPZ_STAGE(4, qo[1], co[1], false, 24u)
                GPZ_STAGE(5, qo[2], co[2], false, 24u)
#undef GPZ_STAGE
                default: {
                    uint32_t q[ITEMS];
                    float x[ITEMS];
                    load_block<ITEMS, FULL>(a.x[f], base, nb, lane, x);
                    c = quantize_field<ITEMS, FULL>(x, nb, lane, a.inv[f], a.twoeb[f], a.eb[f], q);
                    wide = wide || c.wide;
                    stage_codes<ITEMS, false>(q, width, c.clean, mine, vmax, no);
                    break;
                }
            }
            if (!section(f, c, key, width, vmax, no)) break;
        }
    }
    if (!over && pend) {
        wave_lds_sync();
        copy_out<ITEMS>(pend, pend_dst, stage, lane);
        wave_lds_sync();
    }

    if (!SINGLE && wide) {
        defer_block<FORM>(a, b, lane);
        return;
    }
    const bool raw = over || pos >= cap;
    if (raw) {
        // Raw form: the block's floats verbatim, field-major, input order.
        // The barrier orders these stores after the coded ones they replace.
        __syncthreads();
        if (lane == 0) rec[0] = 1u;
        for (uint32_t f = 0; f < F; f++) {
            const float* xf = a.x[f] + base;
            uint32_t* dst = rec + 1 + f * nb;
            for (uint32_t i = lane; i < nb; i += 64) dst[i] = f2u(xf[i]);
        }
    }
    if (SINGLE) {
        place_record(a, b, rec, raw ? cap : pos, lane);
    }
    if (a.perm) {
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            uint32_t p = lane * ITEMS + j;
            if (FULL || p < nb)
                a.perm[base + p] = (uint32_t)(base + (raw ? p : index_of<ITEMS>(kv[j])));
        }
    }
    if (!SINGLE) finish_block<FORM>(a, b, raw ? cap : pos, lane);
}


// Three-step compaction: one workgroup per block, block index = workgroup
// index.  Full blocks take the path without bounds checks, the partial last
// block (if any) the checked one.
template <int ITEMS, int FORM>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void encode_blocks(EncodeArgs a) {
    constexpr uint32_t B = 64 * ITEMS;
    static_assert(FORM != kPlaces, "the lean form copies records");
    __shared__ EncodeSmem<ITEMS> sm;
    const uint32_t b = blockIdx.x;
    if constexpr (FORM == kFew) start_few(a, b);
    const uint64_t left = a.n - (uint64_t)b * B;
    if (left >= B) encode_block<ITEMS, true, false, 3, FORM>(a, b, B, sm.buf);
    else encode_block<ITEMS, false, false, 3, FORM>(a, b, (uint32_t)left, sm.buf);
}

// The same with no early fields beside the key fields (EARLY = 0) and the
// sort's lean scan: at most 168 VGPRs, three waves per SIMD instead of two
// (four below B = 1024, where 103 VGPRs and 9 KB of LDS allow it).  Up to
// B = 1024 this is faster on every workload measured: the late fields' loads
// are hidden by the additional wave (B = 1024: cosmology 64M x 6 -4 %, md
// 32M x 6 -4 %, LiDAR 100M x 3 -13 %; B = 512, cosmology 4M x 6: 72 -> 62 us,
// B = 256 within 1 %).  At B = 2048 both spill.
template <int ITEMS>
constexpr bool kLean = ITEMS <= 16;
template <int ITEMS>
constexpr int kWaves = ITEMS == 16 ? 3 : ITEMS < 16 ? 4 : 2;

template <int ITEMS, int FORM>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kWaves<ITEMS>))) void encode_blocks_lean(EncodeArgs a) {
    constexpr uint32_t B = 64 * ITEMS;
    __shared__ EncodeSmem<ITEMS> sm;
    uint32_t b = blockIdx.x;
    if constexpr (FORM == kPlaces) {
        const Role r = role_of(a, b);
        if (r.idle) return;
        if (!r.encode) {
            place_records(a, r.super, r.part, threadIdx.x);
            return;
        }
        b = r.block;
    }
    if constexpr (FORM == kFew) start_few(a, b);
    const uint64_t left = a.n - (uint64_t)b * B;
    if (left >= B) encode_block<ITEMS, true, false, 0, FORM>(a, b, B, sm.buf);
    else encode_block<ITEMS, false, false, 0, FORM>(a, b, (uint32_t)left, sm.buf);
}

// Single-pass compaction: blocks are numbered by a ticket taken when the
// workgroup starts, so a block only ever waits on blocks already running.
template <int ITEMS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void encode_blocks_single(EncodeArgs a) {
    constexpr uint32_t B = 64 * ITEMS;
    __shared__ EncodeSmem<ITEMS> sm;
    uint32_t t = 0;
    if (threadIdx.x == 0) t = atomicAdd(a.ticket, 1u);
    const uint32_t b = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
    const uint64_t left = a.n - (uint64_t)b * B;
    if (left >= B) encode_block<ITEMS, true, true>(a, b, B, sm.buf);
    else encode_block<ITEMS, false, true>(a, b, (uint32_t)left, sm.buf);
}

// Single pass, a snapshot with no particles: header only.
__global__ __launch_bounds__(64) void empty_stream(EncodeArgs a) {
    publish_size(a, 4 * a.prefix, threadIdx.x);
}

template <int ITEMS>
void launch_encode_items(const EncodeArgs& a, bool single_pass, hipStream_t s) {
    if (single_pass) {
        if (a.nblocks) hipLaunchKernelGGL(encode_blocks_single<ITEMS>, dim3(a.nblocks), dim3(64), 0, s, a);
        else hipLaunchKernelGGL(empty_stream, dim3(1), dim3(64), 0, s, a);
        return;
    }
    // one launch: full blocks take the path without bounds checks, a partial
    // last block the checked one, alongside them (not in a second launch
    // that would wait for the first)
    if (a.nblocks == 0) return;
    const dim3 grid(encode_grid(a)), block(64);
    if constexpr (kLean<ITEMS>) {
        if (a.sup) hipLaunchKernelGGL((encode_blocks_lean<ITEMS, kPlaces>), grid, block, 0, s, a);
        else if (a.few) hipLaunchKernelGGL((encode_blocks_lean<ITEMS, kFew>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((encode_blocks_lean<ITEMS, kPlain>), grid, block, 0, s, a);
    } else {
        if (a.few) hipLaunchKernelGGL((encode_blocks<ITEMS, kFew>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((encode_blocks<ITEMS, kPlain>), grid, block, 0, s, a);
    }
}

// Persistent encoder over the full blocks of many snapshots: each wave takes
// `tile` consecutive blocks from a device work queue until it is empty.
template <int ITEMS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void encode_batch(const EncodeArgs* __restrict__ jobs,
                                                   const BatchLaunch* __restrict__ L) {
    constexpr uint32_t B = 64 * ITEMS;
    __shared__ EncodeSmem<ITEMS> sm;
    const uint32_t total = L->total_full, njobs = L->njobs, tile = L->tile;
    const uint32_t* prefix = L->full_prefix;
    for (;;) {
        uint32_t item = 0;
        if (threadIdx.x == 0) item = atomicAdd(L->counter, tile);
        item = (uint32_t)__builtin_amdgcn_readfirstlane((int)item);
        if (item >= total) break;
        const uint32_t end = min(item + tile, total);
        for (uint32_t g = item; g < end; g++) {
            const uint32_t j = find_job(prefix, njobs, g);
            encode_block<ITEMS, true, false>(jobs[j], g - prefix[j], B, sm.buf);
            __syncthreads();
        }
    }
}

// Direct form of encode_batch: one workgroup per block of the batch's
// capacity; workgroups past the bound jobs' blocks exit at once.  No loop
// around the block, so the compiler keeps the register budget of the plain
// kernel.  Up to B = 1024 the partial last blocks of the snapshots take their
// checked path in the same launch (as in the plain form); at B = 2048 that
// path would add spills to every block, so they go to encode_batch_tails.
template <int ITEMS>
constexpr bool kDirectTails = ITEMS <= 16;

template <int ITEMS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kWaves<ITEMS>))) void encode_batch_direct(
    const EncodeArgs* __restrict__ jobs, const BatchLaunch* __restrict__ L) {
    constexpr uint32_t B = 64 * ITEMS;
    constexpr int EARLY = kLean<ITEMS> ? 0 : 3;
    __shared__ EncodeSmem<ITEMS> sm;
    const uint32_t g = blockIdx.x;
    if (g >= (kDirectTails<ITEMS> ? L->total_blocks : L->total_full)) return;
    const uint32_t* prefix = kDirectTails<ITEMS> ? L->block_prefix : L->full_prefix;
    const uint32_t j = find_job(prefix, L->njobs, g);
    const EncodeArgs& a = jobs[j];
    const uint32_t b = g - prefix[j];
    if constexpr (kDirectTails<ITEMS>) {
        const uint64_t left = a.n - (uint64_t)b * B;
        if (left < B) {
            encode_block<ITEMS, false, false, EARLY>(a, b, (uint32_t)left, sm.buf);
            return;
        }
    }
    encode_block<ITEMS, true, false, EARLY>(a, b, B, sm.buf);
}

// The partial last block of each snapshot that has one.
template <int ITEMS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kWaves<ITEMS>))) void encode_batch_tails(const EncodeArgs* __restrict__ jobs,
                                                         const BatchLaunch* __restrict__ L) {
    constexpr uint32_t B = 64 * ITEMS;
    __shared__ EncodeSmem<ITEMS> sm;
    const uint32_t ntail = L->ntail;
    for (uint32_t t = blockIdx.x; t < ntail; t += gridDim.x) {
        const EncodeArgs& a = jobs[__builtin_amdgcn_readfirstlane((int)L->tail_jobs[t])];
        const uint32_t b = a.nblocks - 1;
        const uint32_t nb = (uint32_t)(a.n - (uint64_t)b * B);
        encode_block<ITEMS, false, false, kLean<ITEMS> ? 0 : 3>(a, b, nb, sm.buf);
        __syncthreads();
    }
}

template <int ITEMS>
void launch_encode_batch_items(const EncodeArgs* jobs, const BatchLaunch* L, const BatchShape& S,
                               hipStream_t s) {
    if (S.grid) {
        hipLaunchKernelGGL(encode_batch<ITEMS>, dim3(S.grid), dim3(64), 0, s, jobs, L);
        hipLaunchKernelGGL(encode_batch_tails<ITEMS>, dim3(S.tail_grid), dim3(64), 0, s, jobs, L);
    } else {
        hipLaunchKernelGGL(encode_batch_direct<ITEMS>, dim3(S.direct_grid), dim3(64), 0, s, jobs, L);
        if (!kDirectTails<ITEMS>)
            hipLaunchKernelGGL(encode_batch_tails<ITEMS>, dim3(S.tail_grid), dim3(64), 0, s, jobs, L);
    }
}

}  // namespace

hipError_t launch_encode_batch(const EncodeArgs* jobs, const BatchLaunch* L, const BatchShape& S,
                               hipStream_t s) {
    switch (S.B) {
        case 256: launch_encode_batch_items<4>(jobs, L, S, s); break;
        case 512: launch_encode_batch_items<8>(jobs, L, S, s); break;
        case 1024: launch_encode_batch_items<16>(jobs, L, S, s); break;
        case 2048: launch_encode_batch_items<32>(jobs, L, S, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_encode(const EncodeArgs& a, bool single_pass, hipStream_t s) {
    switch (a.B) {
        case 256: launch_encode_items<4>(a, single_pass, s); break;
        case 512: launch_encode_items<8>(a, single_pass, s); break;
        case 1024: launch_encode_items<16>(a, single_pass, s); break;
        case 2048: launch_encode_items<32>(a, single_pass, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_encode64(const EncodeArgs& a, hipStream_t s) {
    if (a.B != 1024u) return hipErrorInvalidValue;
    if (a.nblocks == 0) return hipSuccess;
    hipLaunchKernelGGL(encode_blocks64, dim3(encode_grid(a)), dim3(64), 0, s, a);
    return hipGetLastError();
}

}  // namespace gpz
