// Block encoder for float64 fields at B = 1024: one wave64 per block, as
// encode.hip does for float32.  Each field of each block is rounded to
// float32 and quantized by the float32 steps when every finite value is then
// reconstructed within the bound of its double (Sec. 5.1), else from the
// doubles with 64-bit steps (grid indices up to 53 bits).
//
// What bounds it: the doubles are read once (8 bytes a value), and the block's
// chain of LDS round trips and its vector instructions take about twice the
// time of that read.  Fields are loaded "striped" (lane l holds particles
// 256k + 4l + {0..3}, 2 KB of the field per instruction pair), since a lane's
// 16 consecutive doubles would be a cache line of its own; the segment IDs
// pass through LDS once to the blocked order the stable sort needs.  The key
// fields are read and quantized again after the sort (from the caches: their
// codes, up to 64 bits each, would not fit the registers beside it).  Wide codes go through the LDS as two
// 32-bit planes, so the block's LDS stays at 12 KB and twelve blocks share a
// CU.  8M x 6 at a bound float32 meets: 389 us with the generic encoder (four
// waves a block, some forty workgroup barriers), 128 here; at one it does not
// (every field wide): the whole call 707 -> 442 us.
#pragma once

#include "encode_block.h"
#include "generic_block.h"
#include "place.h"

namespace gpz {
namespace {

constexpr int kItems = 16;
constexpr uint32_t kB = 64 * kItems;
constexpr uint32_t kPaddedB = 64 * (kItems + 4);
// LDS words: codes in the padded blocked layout, then the packer's staging
// (1024 values of 53 bits, copied out in steps of 256 words); the sort's
// counters and the run tables reuse the region.
constexpr uint32_t kStage64 = kPaddedB;
constexpr uint32_t kWords64 = kStage64 + (kB * 53 / 32 + 255) / 256 * 256;
static_assert(kWords64 >= kCounterWords && kWords64 >= 2 * kB + 192, "phases fit the region");
static_assert(kWords64 * 4 <= 12288, "twelve blocks share a CU");

// Particle of value j of a lane.
__device__ __forceinline__ uint32_t striped(uint32_t lane, uint32_t j) {
    return 256u * (j / 4) + 4u * lane + (j & 3u);
}

typedef double f64x2 __attribute__((ext_vector_type(2)));

template <bool FULL>
__device__ __forceinline__ void load_striped(const double* __restrict__ x, uint64_t base,
                                             uint32_t nb, uint32_t lane, double (&v)[kItems]) {
    const double* p = x + base;
    if (FULL && ((reinterpret_cast<uintptr_t>(x) & 15u) == 0)) {
        const f64x2* p2 = reinterpret_cast<const f64x2*>(p);
#pragma unroll
        for (int k = 0; k < kItems / 4; k++) {
            const f64x2 t = p2[128 * k + 2 * lane], u = p2[128 * k + 2 * lane + 1];
            v[4 * k] = t.x;
            v[4 * k + 1] = t.y;
            v[4 * k + 2] = u.x;
            v[4 * k + 3] = u.y;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kItems; j++) {
            const uint32_t i = striped(lane, j);
            v[j] = (FULL || i < nb) ? p[i] : 0.0;
        }
    }
}

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
    const uint32_t hi = wave_max_u32((uint32_t)(v >> 32));
    const uint32_t lo = wave_max_u32((uint32_t)(v >> 32) == hi ? (uint32_t)v : 0u);
    return ((uint64_t)hi << 32) | lo;
}

// A field after quantization: the stored minimum's bits, the largest grid
// index, no outliers (clean), 64-bit steps (wide).
struct Field64 {
    uint64_t lo_bits;
    uint64_t qmax;
    bool clean;
    bool wide;
};

// 64-bit steps (Sec. 5.3) about the doubles' finite minimum lo: grid index of
// x, outlier flag in o.
__device__ __forceinline__ uint64_t quantize_wide(double x, double lo, double inv, double twoeb,
                                                  double eb, bool& o) {
    const double t = (x - lo) * inv;
    const bool in = (t >= 0.0) && (t <= kQMaxWide);
    const uint64_t q = in ? (uint64_t)__builtin_rint(t) : 0ull;
    const double xr = __builtin_fma((double)q, twoeb, lo);
    o = !(in && __builtin_fabs(xr - x) < eb);
    return q;
}

// Quantize one field of the block.  Narrow: codes in q (the grid index, or
// 2 * index + outlier when not clean).  Wide: the index's low words in q and
// its high words, the outlier flag at bit 31, in qh.  Codes past the block
// are 0.
//
// The fast path is exact for a field whose every value is finite and meets
// the bound with the float32 steps: it quantizes with rint(t) and tests the
// largest double error and the largest index once (a value that is not
// finite, or out of range, fails one of the two; see quantize_field).  When
// it fails and every value is finite as a float32, some value misses the
// bound, so the field takes the 64-bit steps; otherwise non-finite values are
// outliers and the finite ones decide.
template <bool FULL>
__device__ __forceinline__ Field64 quantize64(const double (&v)[kItems], uint32_t nb, uint32_t lane,
                                              float inv, float twoeb, float eb,
                                              uint32_t (&q)[kItems], uint32_t (&qh)[kItems]) {
    const double eb64 = (double)eb;
    float m = __builtin_inff();
#pragma unroll
    for (int j = 0; j < kItems; j++)
        m = __builtin_elementwise_minimum(
            m, (FULL || striped(lane, j) < nb) ? (float)v[j] : __builtin_inff());
    float lo = 0.0f;
    if (!__any(__builtin_amdgcn_classf(m, 7))) {  // no NaN, no -inf
        m = wave_min_f32(m);
        lo = (m == __builtin_inff() || m == 0.0f) ? 0.0f : m;
        double emax = 0.0;
        float rmax = 0.0f;
#pragma unroll
        for (int j = 0; j < kItems; j++) {
            const bool valid = FULL || striped(lane, j) < nb;
            const float r = __builtin_rintf(((float)v[j] - lo) * inv);
            const float y = __builtin_fmaf(r, twoeb, lo);
            // (an error is NaN only where r is infinite, which rmax keeps)
            emax = fmax(emax, valid ? __builtin_fabs((double)y - v[j]) : 0.0);
            rmax = fmaxf(rmax, valid ? r : 0.0f);
            q[j] = valid ? (uint32_t)r : 0u;
        }
        const uint32_t qmax = wave_max_u32(rmax <= kQMax ? (uint32_t)rmax : 0xFFFFFFFFu);
        if (__all(emax < eb64) && qmax <= 0xFFFFFFu)
            return {d2u((double)lo), qmax, true, false};
    }
    bool finite = true;
#pragma unroll
    for (int j = 0; j < kItems; j++)
        finite = finite && ((!FULL && striped(lane, j) >= nb) || __builtin_isfinite((float)v[j]));
    if (!__all(finite)) {
        // some value is not finite, or not as a float32
        m = __builtin_inff();
        bool bad = false;
#pragma unroll
        for (int j = 0; j < kItems; j++) {
            const bool valid = FULL || striped(lane, j) < nb;
            const float xf = (float)v[j];
            if (valid && __builtin_isfinite(xf)) m = fminf(m, xf);
            bad = bad || (valid && __builtin_isfinite(v[j]) && !__builtin_isfinite(xf));
        }
        m = wave_min_f32(m);
        lo = (m == __builtin_inff() || m == 0.0f) ? 0.0f : m;
        uint32_t mx = 0;
#pragma unroll
        for (int j = 0; j < kItems; j++) {
            const bool valid = FULL || striped(lane, j) < nb;
            const bool fin = __builtin_isfinite(v[j]);
            const float t = ((float)v[j] - lo) * inv;
            const bool in = (t >= 0.0f) && (t <= kQMax);
            const uint32_t qq = in && fin ? (uint32_t)__builtin_rintf(t) : 0u;
            const float y = __builtin_fmaf((float)qq, twoeb, lo);
            bad = bad || (valid && fin && !(in && __builtin_fabs((double)y - v[j]) < eb64));
            q[j] = valid ? (qq << 1) | (fin ? 0u : 1u) : 0u;
            mx = max(mx, valid ? qq : 0u);
        }
        if (!__any(bad)) return {d2u((double)lo), wave_max_u32(mx), false, false};
    }
    uint64_t mk = ~0ull;
#pragma unroll
    for (int j = 0; j < kItems; j++) {
        const bool valid = FULL || striped(lane, j) < nb;
        if (valid && __builtin_isfinite(v[j])) mk = min(mk, okey64(v[j]));
    }
    mk = ~wave_max_u64(~mk);
    double lo64 = mk == ~0ull ? 0.0 : from_okey64(mk);
    if (lo64 == 0.0) lo64 = 0.0;
    const double twoeb64 = 2.0 * eb64, inv64 = 1.0 / twoeb64;
    uint64_t mx = 0;
    bool any = false;
#pragma unroll
    for (int j = 0; j < kItems; j++) {
        const bool valid = FULL || striped(lane, j) < nb;
        bool o;
        uint64_t qq = quantize_wide(v[j], lo64, inv64, twoeb64, eb64, o);
        qq = valid ? qq : 0ull;
        o = o && valid;
        q[j] = (uint32_t)qq;
        qh[j] = (uint32_t)(qq >> 32) | (o ? 0x80000000u : 0u);
        mx = qq > mx ? qq : mx;
        any = any || o;
    }
    return {d2u(lo64), wave_max_u64(mx), !__any(any), true};
}

// One word per particle, striped, into the padded blocked layout at `work`.
__device__ __forceinline__ void put_striped(uint32_t* work, uint32_t lane,
                                            const uint32_t (&q)[kItems]) {
    uint4* const st = reinterpret_cast<uint4*>(work) + lane + lane / (kItems / 4);
#pragma unroll
    for (int k = 0; k < kItems / 4; k++)
        st[k * (64 + 64 / (kItems / 4))] =
            make_uint4(q[4 * k], q[4 * k + 1], q[4 * k + 2], q[4 * k + 3]);
}

// Fixed-length packing of 16 values of a run-time width 24 < w <= 53 or less
// per lane into the staging words at dst (the lane's first word): the same
// segment layout as pack16.  Bit positions inside a lane's segment are the
// same for every lane, so each completed word is stored on a wave-uniform
// branch; for odd w the odd lane's words are shifted by the 16 bits its
// segment starts into a word, and the even lane completes the shared word.
__device__ __forceinline__ void pack_wide(const uint32_t (&lo)[kItems], const uint32_t (&hi)[kItems],
                                          uint32_t w, uint32_t* dst, uint32_t lane) {
    const bool oddw = (w & 1u) != 0u, odd = oddw && (lane & 1u) != 0u;
    const uint32_t shift = odd ? 16u : 0u;
    uint32_t acc = 0u, prev = 0u, first = 0u, k = 0, pos = 0;
    // word k of the lane's segment is complete
    auto flush = [&]() {
        if (k == 0) first = acc;
        const uint32_t word = (uint32_t)((((uint64_t)acc << 32) | prev) >> (32u - shift));
        if (k > 0 || !odd) dst[k] = word;
        prev = acc;
        k++;
    };
    auto append = [&](uint32_t v, uint32_t width) {  // 1 <= width <= 32, uniform
        acc |= v << pos;
        pos += width;
        if (pos >= 32u) {
            flush();
            pos -= 32u;
            acc = pos ? v >> (width - pos) : 0u;
        }
    };
#pragma unroll
    for (int j = 0; j < kItems; j++) {
        if (w <= 32u) {
            append(lo[j], w);
        } else {
            append(lo[j], 32u);
            append(hi[j], w - 32u);
        }
    }
    if (oddw) {
        // 16 bits are left: the even lane completes its word with the odd
        // lane's first 16; the odd lane's last word is whole (w = 1: its
        // only 16 bits are in the shared word)
        if (k == 0) first = acc;
        const uint32_t nxt = dpp<kRowShl1>(first << 16);
        if (k > 0 || !odd) dst[k] = odd ? (acc << 16) | (prev >> 16) : acc | nxt;
    }
}

template <bool FULL>
__device__ __forceinline__ void encode_block64(const EncodeArgs& a, uint32_t b, uint32_t nb,
                                               uint32_t* work) {
    uint32_t* const stage = work + kStage64;
    const uint32_t lane = threadIdx.x;
    const uint64_t base = (uint64_t)b * kB;
    const uint32_t F = a.F, K = a.K, KF = a.KF;
    uint32_t* __restrict__ rec = a.temp + (uint64_t)b * a.slot_words;
    const uint32_t cap = 1 + 2 * F * nb;  // raw record length
    auto field = [&](uint32_t f) { return reinterpret_cast<const double*>(a.x[f].get()); };

    // ---- Stage 1 (Sec. 4.1): key axes, segment IDs accumulated per axis
    // (axis 0 most significant)
    uint32_t kv[kItems];
    uint32_t sk[3] = {0, 0, 0};
#pragma unroll
    for (int j = 0; j < kItems; j++) kv[j] = 0;
    double x[kItems];
    load_striped<FULL>(field(0), base, nb, lane, x);
#pragma unroll 1
    for (uint32_t ax = 0; ax < KF; ax++) {
        uint32_t q[kItems], qh[kItems];
        const Field64 c =
            quantize64<FULL>(x, nb, lane, a.inv[ax], a.twoeb[ax], a.eb[ax], q, qh);
        // (after the last axis, field 0 again: its section comes first)
        load_striped<FULL>(field(ax + 1 < KF ? ax + 1 : 0u), base, nb, lane, x);
        const uint32_t W = bit_width64(c.qmax), s = W > K ? W - K : 0;
        sk[0] = ax == 0 ? s : sk[0];
        sk[1] = ax == 1 ? s : sk[1];
        sk[2] = ax == 2 ? s : sk[2];
        if (c.wide) {
#pragma unroll
            for (int j = 0; j < kItems; j++) {
                const uint64_t v = ((uint64_t)(qh[j] & 0x7FFFFFFFu) << 32) | q[j];
                kv[j] = (kv[j] << K) | (uint32_t)(v >> s);
            }
        } else {
            const uint32_t o0 = c.clean ? 0u : 1u;
#pragma unroll
            for (int j = 0; j < kItems; j++) kv[j] = (kv[j] << K) | (q[j] >> (s + o0));
        }
    }
    uint32_t keyor = 0;
#pragma unroll
    for (int j = 0; j < kItems; j++) keyor |= kv[j];  // (codes past the block are 0)
    keyor = wave_or_u32(keyor);

    // to the blocked order the stable sort needs, through LDS
    put_striped(work, lane, kv);
    wave_lds_sync();
    {
        const uint4* bl = reinterpret_cast<const uint4*>(work + lane * (kItems + 4));
#pragma unroll
        for (int k = 0; k < kItems / 4; k++) {
            const uint4 t = bl[k];
            kv[4 * k] = t.x;
            kv[4 * k + 1] = t.y;
            kv[4 * k + 2] = t.z;
            kv[4 * k + 3] = t.w;
        }
    }
    wave_lds_sync();
#pragma unroll
    for (int j = 0; j < kItems; j++)
        kv[j] = (kv[j] << 16) | (4u * pad_addr<kItems>(lane * kItems + j));

    // ---- Stage 2 (Sec. 4.2): stable in-block sort by segment ID
    const uint32_t keybits = K * KF;
    for (uint32_t sh = 0; sh < keybits; sh += kDigitBits) {
        if (((keyor >> sh) & (kDigits - 1)) == 0) continue;  // identity pass
        radix_pass<kItems, FULL, true>(kv, sh, nb, lane, work, work);
    }

    // ---- Stage 3 (Sec. 4.3): run-length and delta coding of the sorted IDs
    uint32_t* uniq = work;
    uint32_t* start = work + kB;
    const uint32_t U = code_runs<kItems, FULL>(kv, nb, lane, uniq, start);
    uint32_t gv[kItems], cv[kItems];
    run_gaps<kItems>(uniq, U, lane, gv);
    run_counts<kItems>(start, U, lane, cv);
    uint32_t gmax = 0, cmax = 0;
#pragma unroll
    for (int j = 0; j < kItems; j++) {
        gmax = max(gmax, gv[j]);
        cmax = max(cmax, cv[j]);
    }
    const uint32_t w_gap = bit_width(wave_max_u32(gmax));
    const uint32_t w_cnt = bit_width(wave_max_u32(cmax));
    uint32_t pos = 2;
    bool over = false;
    const uint32_t gw = words_for(U, w_gap), cw = words_for(U, w_cnt);
    if (pos + gw + cw > cap) {
        over = true;
    } else {
        wave_lds_sync();  // uniq/start reads done before `work` is reused
        pack_array<kItems>(gv, U, w_gap, rec + pos, stage, lane);
        pack_array<kItems>(cv, U, w_cnt, rec + pos + gw, stage, lane);
        pos += gw + cw;
    }

    // One field's section from its codes (striped; q and, wide, qh): minimum
    // and field word, the codes permuted to sorted order (a key field's low
    // sk bits) and packed, its outliers.  False when the block is stored raw.
    auto section = [&](uint32_t f, const Field64& c, bool key, uint32_t s,
                       const uint32_t (&q)[kItems], const uint32_t (&qh)[kItems]) -> bool {
        const uint32_t o0 = !c.wide && !c.clean ? 1u : 0u;  // outlier flag below the index
        const uint64_t keep = key ? low_mask64(s) : ~0ull;
        const uint32_t keep_lo = (uint32_t)keep, keep_hi = (uint32_t)(keep >> 32) & 0x7FFFFFFFu;
        uint32_t w = bit_width64(c.qmax);
        if (key) {
            uint64_t mx = 0;
#pragma unroll
            for (int j = 0; j < kItems; j++) {
                const uint64_t v = c.wide ? ((uint64_t)(qh[j] & keep_hi) << 32) | (q[j] & keep_lo)
                                          : (uint64_t)((q[j] >> o0) & keep_lo);
                mx = v > mx ? v : mx;
            }
            w = bit_width64(wave_max_u64(mx));
        }
        uint32_t no = 0;
        if (!c.clean) {
#pragma unroll
            for (int j = 0; j < kItems; j++) no += c.wide ? qh[j] >> 31 : q[j] & 1u;
            no = wave_sum_u32(no);
        }
        const uint32_t pw = words_for(nb, w);
        if ((uint64_t)pos + 3 + pw + 3ull * no > cap) return false;
        if (lane == 0) {
            rec[pos] = (uint32_t)c.lo_bits;
            rec[pos + 1] = (uint32_t)(c.lo_bits >> 32);
            rec[pos + 2] = c.wide ? (w | (no << 6) | (1u << 31)) : (w | (no << 5));
        }
        pos += 3;
        wave_lds_sync();
        uint32_t vals[kItems];
        put_striped(work, lane, q);
        wave_lds_sync();
#pragma unroll
        for (int j = 0; j < kItems; j++)
            vals[j] = FULL || lane * kItems + j < nb ? staged_at(work, kv[j]) : 0u;
        if (c.wide) {
            uint32_t high[kItems];
            wave_lds_sync();  // the low words are read before the high ones replace them
            put_striped(work, lane, qh);
            wave_lds_sync();
#pragma unroll
            for (int j = 0; j < kItems; j++) {
                high[j] = FULL || lane * kItems + j < nb ? staged_at(work, kv[j]) & keep_hi : 0u;
                vals[j] &= keep_lo;
            }
            if (w > 0) pack_wide(vals, high, w, stage + ((lane * w) >> 1), lane);
        } else {
            if (key || !c.clean) {
#pragma unroll
                for (int j = 0; j < kItems; j++)
                    vals[j] = __builtin_amdgcn_ubfe(vals[j], o0, key ? s : 24u);
            }
            pack_stage<kItems>(vals, nb, w, stage, lane);
        }
        wave_lds_sync();
        copy_out<kItems>(pw, rec + pos, stage, lane);
        pos += pw;
        if (no) {
            // outlier flags of the lane's sorted positions, from the codes
            // (wide: their high words) still in LDS
            uint32_t flags = 0;
#pragma unroll
            for (int j = 0; j < kItems; j++)
                if (FULL || lane * kItems + j < nb)
                    flags |= ((staged_at(work, kv[j]) >> (c.wide ? 31u : 0u)) & 1u) << j;
            const uint32_t cnt = __builtin_popcount(flags);
            uint32_t k = wave_incl_scan_u32(cnt) - cnt;
            uint32_t* ol = rec + pos;
            const uint64_t* xf = reinterpret_cast<const uint64_t*>(a.x[f].get()) + base;
#pragma unroll 1
            for (int j = 0; j < kItems; j++) {
                if ((flags >> j) & 1u) {
                    // the particle at sorted position lane * 16 + j, from its
                    // place in the permutation (kept in registers: selected
                    // without an indexed array)
                    uint32_t item = 0;
#pragma unroll
                    for (int t = 0; t < kItems; t++) item = t == j ? kv[t] : item;
                    const uint64_t u = xf[index_of<kItems>(item)];
                    ol[3 * k] = lane * kItems + j;
                    ol[3 * k + 1] = (uint32_t)u;
                    ol[3 * k + 2] = (uint32_t)(u >> 32);
                    k++;
                }
            }
            pos += 3 * no;
        }
        return true;
    };

    // every field, the next one fetched while this one is permuted and packed
    bool any_wide = false;
#pragma unroll 1
    for (uint32_t f = 0; f < F && !over; f++) {
#pragma unroll
        for (int j = 0; j < kItems; j++) asm volatile("" : "+v"(kv[j]));
        uint32_t q[kItems], qh[kItems];
        const Field64 c = quantize64<FULL>(x, nb, lane, a.inv[f], a.twoeb[f], a.eb[f], q, qh);
        if (f + 1 < F) load_striped<FULL>(field(f + 1), base, nb, lane, x);
        any_wide = any_wide || c.wide;
        const uint32_t s = f == 0 ? sk[0] : f == 1 ? sk[1] : sk[2];
        if (!section(f, c, f < KF, s, q, qh)) over = true;
    }

    const bool raw = over || pos >= cap;
    if (raw) {
        // raw form: the block's values verbatim, field-major, input order;
        // the barrier orders these stores after the coded ones they replace
        __syncthreads();
        if (lane == 0) rec[0] = 1u;
        for (uint32_t f = 0; f < F; f++) {
            const uint64_t* xf = reinterpret_cast<const uint64_t*>(a.x[f].get()) + base;
            uint32_t* dst = rec + 1 + 2 * f * nb;
            for (uint32_t i = lane; i < nb; i += 64) {
                const uint64_t u = xf[i];
                dst[2 * i] = (uint32_t)u;
                dst[2 * i + 1] = (uint32_t)(u >> 32);
            }
        }
    } else if (lane == 0) {
        rec[0] = (U << 2) | (any_wide ? 1u << 31 : 0u);
        rec[1] = w_gap | (w_cnt << 5) | ((sk[0] & 31u) << 10) | ((sk[1] & 31u) << 15) |
                 ((sk[2] & 31u) << 20) | ((sk[0] >> 5) << 25) | ((sk[1] >> 5) << 26) |
                 ((sk[2] >> 5) << 27);
    }
    if (lane == 0 && !raw && any_wide) atomicOr(a.wide_flag, 1u);
    if (a.perm) {
#pragma unroll
        for (int j = 0; j < kItems; j++) {
            const uint32_t p = lane * kItems + j;
            if (FULL || p < nb)
                a.perm[base + p] = (uint32_t)(base + (raw ? p : index_of<kItems>(kv[j])));
        }
    }
    finish_block<kPlaces>(a, b, raw ? cap : pos, lane);
}

// One workgroup per block; the partial last block takes the checked path.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) void encode_blocks64(EncodeArgs a) {
    __shared__ __align__(16) uint32_t work[kWords64];
    const Role r = role_of(a, blockIdx.x);
    if (r.idle) return;
    if (!r.encode) {
        place_records(a, r.super, r.part, threadIdx.x);
        return;
    }
    const uint32_t b = r.block;
    const uint64_t left = a.n - (uint64_t)b * kB;
    if (left >= kB) encode_block64<true>(a, b, kB, work);
    else encode_block64<false>(a, b, (uint32_t)left, work);
}

}  // namespace
}  // namespace gpz
