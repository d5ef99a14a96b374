// Compaction (Sec. 4.4, steps two and three): a device-level exclusive scan
// of the block record lengths, then a copy of every record to its final
// offset together with the stream header and tables.  Also: a fill kernel
// (used instead of hipMemset so the sequence stays graph-capturable), the
// error-bound check and the per-field range reduction.
#include <atomic>

#include "copy_record.h"

namespace gpz {
namespace {

constexpr uint32_t kScanThreads = 1024;

__global__ __launch_bounds__(kScanThreads) void scan_lengths(ScanArgs a) {
    __shared__ uint64_t part[kScanThreads];
    scan_superblocks<kScanThreads>(a, part);
}

__global__ __launch_bounds__(kScanThreads) void scan_lengths_batch(const ScanArgs* jobs,
                                                                    const BatchLaunch* L) {
    __shared__ uint64_t part[kScanThreads];
    const uint32_t njobs = L->njobs;
    for (uint32_t j = blockIdx.x; j < njobs; j += gridDim.x) {
        scan_superblocks<kScanThreads>(jobs[j], part);
        __syncthreads();
    }
}

// One wave per block record: copy it from its slot to its final offset
// (superblock offset + lengths of the earlier blocks of the superblock).
// Nothing is written when the stream does not fit the output buffer.
__device__ __forceinline__ void copy_body(const CopyArgs& a, uint32_t b, uint32_t lane) {
    const uint64_t total = *a.total_bytes;
    if (total > a.capacity) return;
    const uint32_t sb = b / kSuper, first = sb * kSuper;
    const uint32_t before = wave_sum_u32(first + lane < b ? a.lens[first + lane] : 0u);
    place_record(a, b, a.lens[b], a.supoff[sb] + before, lane);
}

template <bool FEW>
__global__ __launch_bounds__(256) void copy_records(CopyArgs a) {
    const uint32_t b = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (b >= a.nblocks) return;
    if (FEW && !any_left(a.left, a.nblocks)) return;  // finish_few placed the records
    copy_body(a, b, threadIdx.x & 63u);
}

// After an encoder that copied records itself (place.h): one workgroup per
// part of the superblocks it was to copy, which normally finds its flag set
// and exits, then one wave per block of the rest.  Four waves a part: with
// every block left for 64-bit steps (8M x 6 at a relative bound of 1e-8, where
// all records are copied here) the call took 1288 us at one wave a part, 1228
// at two, 1208 at four, 1207 at eight; cosmology 64M x 6, where nearly all
// workgroups exit, 516.7, 518.5, 519.5, 519.6.
constexpr uint32_t kRestWaves = 4;
__global__ __launch_bounds__(64 * kRestWaves) void copy_rest(CopyArgs a) {
    constexpr uint32_t kEach = kSuper / kPlaceParts, kOwn = kEach / kRestWaves;
    const uint32_t parts = a.placed * kPlaceParts, g = blockIdx.x;
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    if (g >= parts) {
        const uint32_t b = a.placed * kSuper + (g - parts) * kRestWaves + wave;
        if (b < a.nblocks) copy_body(a, b, lane);
        return;
    }
    if ((a.copied[g / kPlaceParts] >> (g % kPlaceParts)) & 1u) return;
    for (uint32_t i = 0; i < kOwn; i++) copy_body(a, g * kEach + wave * kOwn + i, lane);
}

// Direct form: one wave per block of the batch's capacity (4 per
// workgroup), as the plain copy; waves past the bound jobs' blocks exit.
__global__ __launch_bounds__(256) void copy_records_batch_direct(const CopyArgs* jobs,
                                                                 const BatchLaunch* L) {
    const uint32_t g = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (g >= L->total_blocks) return;
    const uint32_t* prefix = L->block_prefix;
    const uint32_t j = find_job(prefix, L->njobs, g);
    copy_body(jobs[j], g - prefix[j], threadIdx.x & 63u);
}

__global__ __launch_bounds__(256) void copy_records_batch(const CopyArgs* jobs,
                                                          const BatchLaunch* L) {
    const uint32_t total = L->total_blocks, njobs = L->njobs;
    const uint32_t* prefix = L->block_prefix;
    for (uint32_t g = blockIdx.x * 4 + (threadIdx.x >> 6); g < total; g += gridDim.x * 4) {
        const uint32_t j = find_job(prefix, njobs, g);
        copy_body(jobs[j], g - prefix[j], threadIdx.x & 63u);
    }
}

// Accumulators of the reporting calls in one launch: nzero words of zeros,
// and nkeys minimum then nkeys maximum range keys at their identities.
__global__ __launch_bounds__(256) void reset_stats(uint32_t* zero, uint32_t nzero, int* keys,
                                                   uint32_t nkeys) {
    for (uint32_t i = threadIdx.x; i < nzero; i += 256) zero[i] = 0u;
    for (uint32_t i = threadIdx.x; i < nkeys; i += 256) {
        keys[i] = 0x7FFFFFFF;
        keys[nkeys + i] = (int)0x80000000;
    }
}

__global__ void fill_u32(uint32_t* p, uint32_t value, uint64_t count) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = value;
}

__global__ __launch_bounds__(256) void copy_words(uint32_t* dst, const uint32_t* src,
                                                  uint32_t words) {
    for (uint32_t i = threadIdx.x; i < words; i += 256) dst[i] = src[i];
}

struct BoundArgs {
    const float* orig[kMaxFields];
    const float* recon[kMaxFields];
    float eb[kMaxFields];
    const uint32_t* perm;
    uint64_t n;
    uint32_t F;
    unsigned long long* viol;
    unsigned long long* maxerr_bits;
    double* sumsq;  // STATS: sum of squared differences per field
    int* keys;      // STATS: range keys of the originals, [0, F) minima, [F, 2F) maxima
};

// Order-preserving map of float bits to signed integers (-0 < +0).
__device__ __forceinline__ int order_key(float v) {
    int i = __float_as_int(v);
    return i ^ ((i >> 31) & 0x7FFFFFFF);
}

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
__device__ __forceinline__ double wave_max_f64(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}

// 16 bytes at 4-byte alignment (the hardware takes unaligned vector loads).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

constexpr uint32_t kCheckChunk = 1024;  // positions per wave step
constexpr int kCheckItems = kCheckChunk / 64;
// Two workgroups of eight waves per CU: 128 registers let four waves share a SIMD, whose loads
// (8 KB each) cover the memory's latency without a prefetch (with one, which
// spilled at this occupancy, a whole 16M x 6 report took 295 us; 238 without).
// Eight waves share a workgroup's atomics at the end, which run one after the
// other on a field's words: 128 us at 16M x 6, with four waves 141, with
// sixteen 128 (and fewer CUs at work on a small snapshot).
constexpr uint32_t kCheckWaves = 8;
constexpr uint32_t kCheckGroups = 2;

// Values 256k + 4 lane + e of a chunk that starts at p (whole, or those whose
// bit is set in `live`; the others are 0).
__device__ __forceinline__ void check_load(const float* p, bool whole, uint32_t live, uint32_t lane,
                                           float (&v)[kCheckItems]) {
    if (whole) {
#pragma unroll
        for (int k = 0; k < kCheckItems / 4; k++) {
            const f32x4u t = __builtin_nontemporal_load(
                reinterpret_cast<const f32x4u*>(p + 256 * k + 4 * lane));
            v[4 * k] = t.x;
            v[4 * k + 1] = t.y;
            v[4 * k + 2] = t.z;
            v[4 * k + 3] = t.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kCheckItems; j++) {
            const uint32_t i = 256u * (j / 4) + 4u * lane + (j & 3u);
            v[j] = (live >> j) & 1u ? p[i] : 0.0f;
        }
    }
}

// Error-bound verification, with STATS also the sum of squared errors and the
// finite range of the originals.  Each wave takes chunks of 1024 positions.
// A field's originals in the chunk's own window come in with 16-byte loads
// and are gathered through LDS, because a GPZ permutation is block-local (an
// entry outside the window is read from memory, one outside [0, n) counts as
// a violation and is not read); the same registers give the originals'
// range, so they are read once.  A pair passes when its bits match or |recon - orig|
// <= eb in double.
//
// The bound is the read of both arrays (and of the permutation once for all
// fields), so the per-value work is kept to five double operations: the
// largest error, the finite range and the presence of a NaN are tested once
// per lane and chunk (a lane's sum is NaN exactly when one of its differences
// is), and only chunks that fail a test count pairs one by one or reduce
// across the wave.  16M x 6 with a permutation (0.83 GB): 128 us, 6.5 TB/s;
// the check that gathered the originals from memory took 274 us and the
// separate range pass another 100.
template <bool STATS>
__global__ __launch_bounds__(64 * kCheckWaves) __attribute__((amdgpu_waves_per_eu(4))) void bound_check_kernel(BoundArgs a) {
    __shared__ __align__(16) float win[kCheckWaves][kCheckChunk];  // stored 16 bytes at a time
    __shared__ double sm[kCheckWaves][kMaxFields], ss[kCheckWaves][kMaxFields];
    __shared__ unsigned long long sv[kCheckWaves][kMaxFields];
    __shared__ int skn[kCheckWaves][kMaxFields], skx[kCheckWaves][kMaxFields];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    float* const mywin = win[w];
    sm[w][lane] = 0.0;
    ss[w][lane] = 0.0;
    sv[w][lane] = 0;
    skn[w][lane] = 0x7FFFFFFF;
    skx[w][lane] = (int)0x80000000;
    wave_lds_sync();
    const uint64_t nchunks = (a.n + kCheckChunk - 1) / kCheckChunk;
    for (uint64_t c = (uint64_t)blockIdx.x * kCheckWaves + w; c < nchunks;
         c += (uint64_t)gridDim.x * kCheckWaves) {
        const uint64_t c0 = c * kCheckChunk;
        const uint64_t left = a.n - c0;
        const bool whole = left >= kCheckChunk;
        // (opaque: no 64-bit index per position is kept across the chunks)
        uint32_t ln = lane;
        asm volatile("" : "+v"(ln));
        // position of each pair's original: its offset in the window, or
        // (bit set in `far`) elsewhere
        uint32_t src[kCheckItems];
        uint32_t live = 0xFFFFu, far = 0u;
        if (whole && a.perm) {
#pragma unroll
            for (int k = 0; k < kCheckItems / 4; k++) {
                const u32x4u t =
                    *reinterpret_cast<const u32x4u*>(a.perm + c0 + 256 * k + 4 * ln);
                src[4 * k] = t.x - (uint32_t)c0;
                src[4 * k + 1] = t.y - (uint32_t)c0;
                src[4 * k + 2] = t.z - (uint32_t)c0;
                src[4 * k + 3] = t.w - (uint32_t)c0;
            }
        } else {
#pragma unroll
            for (int j = 0; j < kCheckItems; j++) {
                const uint32_t i = 256u * (j / 4) + 4u * ln + (j & 3u);
                src[j] = i;
                if (i >= left) live &= ~(1u << j);
                else if (a.perm) src[j] = a.perm[c0 + i] - (uint32_t)c0;
            }
        }
        // (past 2^32 the 32-bit entries never name the chunk's own window)
        const uint32_t inwin = a.perm && (c0 >> 32) ? 0u
                               : whole ? kCheckChunk : (uint32_t)left;
#pragma unroll
        for (int j = 0; j < kCheckItems; j++)
            if (src[j] >= inwin) far |= 1u << j;
        far &= live;
        const bool plain = !__any(far != 0u || live != 0xFFFFu);
        for (uint32_t f = 0; f < a.F; f++) {
            // (opaque: the compiler would keep a lane mask per bit, and spill
            // them, across the loop over fields)
            asm volatile("" : "+v"(live), "+v"(far));
            float xn[kCheckItems], x[kCheckItems], y[kCheckItems];
            check_load(a.orig[f] + c0, whole, live, ln, xn);
            check_load(a.recon[f] + c0, whole, live, ln, y);
            if (a.perm) {
#pragma unroll
                for (int k = 0; k < kCheckItems / 4; k++)
                    reinterpret_cast<float4*>(mywin)[64 * k + ln] =
                        make_float4(xn[4 * k], xn[4 * k + 1], xn[4 * k + 2], xn[4 * k + 3]);
            }
            if (STATS) {
                // finite range of the window: a lane whose plain minimum or
                // maximum is NaN or infinite filters its values one by one
                float mn = xn[0], mx = xn[0];
#pragma unroll
                for (int j = 1; j < kCheckItems; j++) {
                    mn = __builtin_elementwise_minimum(mn, xn[j]);
                    mx = __builtin_elementwise_maximum(mx, xn[j]);
                }
                int kn = order_key(mn), kx = order_key(mx);
                if (!whole || __any(!__builtin_isfinite(mn) || !__builtin_isfinite(mx))) {
                    kn = 0x7FFFFFFF;
                    kx = (int)0x80000000;
#pragma unroll
                    for (int j = 0; j < kCheckItems; j++) {
                        if (((live >> j) & 1u) && __builtin_isfinite(xn[j])) {
                            kn = min(kn, order_key(xn[j]));
                            kx = max(kx, order_key(xn[j]));
                        }
                    }
                }
                if (__any(kn < skn[w][f] || kx > skx[w][f])) {
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) {
                        kn = min(kn, __shfl_xor(kn, o));
                        kx = max(kx, __shfl_xor(kx, o));
                    }
                    if (lane == 0) {
                        skn[w][f] = min(kn, skn[w][f]);
                        skx[w][f] = max(kx, skx[w][f]);
                    }
                }
            }
            if (a.perm) {
                wave_lds_sync();
#pragma unroll
                for (int j = 0; j < kCheckItems; j++) x[j] = mywin[src[j] & (kCheckChunk - 1u)];
                wave_lds_sync();  // gathered before the next field's window replaces it
            } else {
#pragma unroll
                for (int j = 0; j < kCheckItems; j++) x[j] = xn[j];
            }
            const double eb = (double)a.eb[f];
            double m = 0.0, q = 0.0;
            bool exact = plain;
            if (plain) {
#pragma unroll
                for (int j = 0; j < kCheckItems; j++) {
                    const double d = __builtin_fabs((double)y[j] - (double)x[j]);
                    m = fmax(m, d);
                    q = __builtin_fma(d, d, q);
                }
                exact = !__any(!(m <= eb) || __builtin_isnan(q));
            }
            if (!exact) {
                unsigned long long v = 0;
                m = 0.0;
                q = 0.0;
#pragma unroll
                for (int j = 0; j < kCheckItems; j++) {
                    if (!((live >> j) & 1u)) continue;
                    float xo = x[j];
                    // (opaque: neither the differences above nor a 64-bit
                    // address per position are kept for this path)
                    uint32_t at = src[j] + (uint32_t)c0;
                    asm volatile("" : "+v"(xo), "+v"(at));
                    if ((far >> j) & 1u) {
                        if (at >= a.n) {  // not a permutation of [0, n)
                            v++;
                            continue;
                        }
                        xo = a.orig[f][at];
                    }
                    const double d = __builtin_fabs((double)y[j] - (double)xo);
                    if (!__builtin_isnan(d)) {
                        m = fmax(m, d);
                        q = __builtin_fma(d, d, q);
                    }
                    if (f2u(xo) != f2u(y[j]) && !(d <= eb)) v++;
                }
                v = wave_sum_u64(v);
                if (lane == 0) sv[w][f] += v;
            }
            if (__any(m > sm[w][f])) {
                m = wave_max_f64(m);
                if (lane == 0) sm[w][f] = fmax(m, sm[w][f]);
            }
            if (STATS) {
                q = wave_sum_f64(q);
                if (lane == 0) ss[w][f] += q;
            }
            wave_lds_sync();
        }
    }
    __syncthreads();
    for (uint32_t f = threadIdx.x; f < a.F; f += 64 * kCheckWaves) {
        unsigned long long tv = 0;
        double tm = 0.0, tq = 0.0;
        int kn = 0x7FFFFFFF, kx = (int)0x80000000;
        for (uint32_t i = 0; i < kCheckWaves; i++) {
            tv += sv[i][f];
            tm = fmax(tm, sm[i][f]);
            tq += ss[i][f];
            kn = min(kn, skn[i][f]);
            kx = max(kx, skx[i][f]);
        }
        if (tv) atomicAdd(&a.viol[f], tv);
        if (tm > 0.0) atomicMax(&a.maxerr_bits[f], (unsigned long long)__double_as_longlong(tm));
        if (STATS) {
            if (tq != 0.0) atomicAdd(&a.sumsq[f], tq);
            if (kn <= kx) {
                atomicMin(&a.keys[f], kn);
                atomicMax(&a.keys[a.F + f], kx);
            }
        }
    }
}

// Structure statistics of a stream: outliers per field (coded blocks) and
// raw blocks.  One lane per block, one wave per superblock: the record offset
// is the superblock's plus an exclusive scan of the lengths across the wave
// (each lane summing the lengths before its own took as long as the walk);
// the lane walks the record's array headers, one dependent read per field,
// which is what bounds it.  Malformed structure sets *err.
struct StatsArgs {
    const uint32_t* in;
    uint64_t in_words;
    uint64_t n;
    uint32_t F, B, nblocks;
    uint64_t prefix;
    unsigned long long* outliers;  // F
    unsigned long long* raw;
    uint32_t* err;
};

__global__ __launch_bounds__(256) void stream_stats_kernel(StatsArgs a) {
    // A call starts with the default block size: on a stream of another one (or
    // of another shape, which the host finds in the header) nothing is walked.
    // 32M particles at B = 256: the call 59 us with the walk, 44 without, 60 with
    // the header fetched first.
    if (a.in[4] != a.F || a.in[5] != a.B || a.in[7] != a.nblocks) return;
    const uint32_t b = blockIdx.x * 256 + threadIdx.x;
    const bool live = b < a.nblocks;
    const uint64_t nsup = nsuper_of(a.nblocks);
    const uint32_t* sup = a.in + kHeaderWords;
    const uint32_t* lt = sup + 2 * nsup + a.F;
    const uint64_t rec_total = a.in_words - a.prefix;
    const uint32_t vw = (a.in[1] >> 16) & 1u ? 2u : 1u;  // words per value (float64 stream: 2)
    bool bad = false, raw = false;
    uint64_t off = 0, pos = 0;
    uint32_t len = 0, nn = 0;
    const uint32_t* rec = a.in + a.prefix;
    static_assert(kSuper == 64, "one wave per superblock");
    len = live ? lt[b] : 0u;
    uint64_t before = len;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t t = __shfl_up(before, o);
        before += (threadIdx.x & 63u) >= (uint32_t)o ? t : 0ull;
    }
    before -= len;
    if (live) {
        // superblock entry checked before use, lengths summed in 64 bits (at
        // most 63 of them): no sum wraps, an accepted record lies inside the
        // record area
        const uint32_t sb = b / kSuper;
        const uint64_t sup_off = (uint64_t)sup[2 * sb] | ((uint64_t)sup[2 * sb + 1] << 32);
        off = sup_off + before;
        nn = (uint32_t)((uint64_t)(b + 1) * a.B <= a.n ? a.B : a.n - (uint64_t)b * a.B);
        bad = len < 1 || sup_off > rec_total || off > rec_total || (uint64_t)len > rec_total - off;
        if (!bad) {
            rec += off;
            raw = (rec[0] & 3u) == 1u;
            if (raw) {
                bad = len != 1 + a.F * nn * vw;
            } else {
                bad = len < 2;
                if (!bad) {
                    const uint32_t U = (rec[0] & 0x7FFFFFFFu) >> 2, h1 = rec[1];
                    pos = 2 + (uint64_t)words_for(U, h1 & 31u) + words_for(U, (h1 >> 5) & 31u);
                }
            }
        }
    }
    const bool walk = live && !bad && !raw;
    for (uint32_t f = 0; f < a.F; f++) {
        uint32_t nout = 0;
        if (walk && !bad) {
            if (pos + vw + 1 > len) {
                bad = true;
            } else {
                // field word: w | nout << 5, or w | nout << 6 | 1 << 31 (wide)
                const uint32_t wn = rec[pos + vw];
                const bool wide = (wn >> 31) != 0;
                const uint32_t w = wide ? (wn & 63u) : (wn & 31u);
                nout = wide ? ((wn >> 6) & 0x1FFFFFFu) : ((wn >> 5) & 0x3FFFFFFu);
                pos += vw + 1 + (uint64_t)words_for(nn, w) + (uint64_t)(1 + vw) * nout;
            }
        }
        const uint32_t tot = wave_sum_u32(nout);
        if ((threadIdx.x & 63u) == 0 && tot) atomicAdd(&a.outliers[f], (unsigned long long)tot);
    }
    if (walk && !bad && pos != len) bad = true;
    const uint32_t nraw = wave_sum_u32(live && !bad && raw ? 1u : 0u);
    if ((threadIdx.x & 63u) == 0 && nraw) atomicAdd(a.raw, (unsigned long long)nraw);
    if (live && bad) *a.err = 1u;
}

struct RangeArgs {
    const float* x[kMaxFields];
    uint64_t n;
    uint32_t F;
    uint64_t cpf;  // chunks per field: ceil((n / 4) / (U * 256))
    int* keys;     // order-preserving integer keys: [0, F) minima, [F, 2F) maxima
};

__device__ __forceinline__ void range_take(float v, int& mn, int& mx) {
    if (__builtin_isfinite(v)) {
        const int k = order_key(v);
        mn = min(mn, k);
        mx = max(mx, k);
    }
}

__device__ __forceinline__ void range_take4(const f32x4& v, int& mn, int& mx) {
    range_take(v.x, mn, mx);
    range_take(v.y, mn, mx);
    range_take(v.z, mn, mx);
    range_take(v.w, mn, mx);
}

// Workgroup minimum / maximum of the keys, then one atomic pair per
// workgroup (atomics of many waves on the same few words serialize).  Every
// lane calls it (a change of field is workgroup-uniform).
__device__ __forceinline__ void range_flush(const RangeArgs& a, uint32_t f, int mn, int mx,
                                            int* smin, int* smax) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        mn = min(mn, __shfl_xor(mn, o));
        mx = max(mx, __shfl_xor(mx, o));
    }
    if ((threadIdx.x & 63u) == 0) {
        smin[threadIdx.x >> 6] = mn;
        smax[threadIdx.x >> 6] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < 4; k++) {
            mn = min(mn, smin[k]);
            mx = max(mx, smax[k]);
        }
        if (mn != 0x7FFFFFFF) atomicMin(&a.keys[f], mn);
        if (mx != (int)0x80000000) atomicMax(&a.keys[a.F + f], mx);
    }
    __syncthreads();
}

// Chunk c of the flattened (field, chunk) space: its field, the 16-byte
// vectors of that field past its unaligned head, and the chunk's first vector.
struct RangeChunk {
    uint32_t f;
    const f32x4* xv;
    uint64_t nv, v0;
};

__device__ __forceinline__ RangeChunk range_chunk(const RangeArgs& a, uint64_t c, uint64_t chunk) {
    RangeChunk r;
    r.f = (uint32_t)(c / a.cpf);
    const float* x = a.x[r.f];
    const uint64_t head = ((16u - (reinterpret_cast<uintptr_t>(x) & 15u)) & 15u) / 4u;
    const uint64_t h = head < a.n ? head : a.n;
    r.nv = (a.n - h) / 4;
    r.xv = reinterpret_cast<const f32x4*>(x + h);
    r.v0 = (c - (uint64_t)r.f * a.cpf) * chunk;
    return r;
}

template <int U>
__device__ __forceinline__ void range_load(const RangeChunk& r, uint64_t chunk, f32x4 (&v)[U]) {
    const uint64_t i0 = r.v0 + threadIdx.x;
    if (r.v0 + chunk <= r.nv) {
#pragma unroll
        for (int k = 0; k < U; k++) v[k] = __builtin_nontemporal_load(r.xv + i0 + 256 * k);
    } else {
        const f32x4 nan4 = {__builtin_nanf(""), __builtin_nanf(""), __builtin_nanf(""),
                            __builtin_nanf("")};
#pragma unroll
        for (int k = 0; k < U; k++)
            v[k] = i0 + 256 * k < r.nv ? __builtin_nontemporal_load(r.xv + i0 + 256 * k) : nan4;
    }
}

// Field range over finite values.  The 16-byte vectors of every field are cut
// into chunks of U * 256 vectors (chunk c belongs to field c / cpf);
// every workgroup takes a contiguous range of them, so that it ends one field,
// rarely two, and each field's keys see few of the workgroups' atomics, which
// run one after the other (with chunks g, g + gridDim.x, ... every workgroup
// ended every field: 1M x 6 took 43 us for 24 MB, 17 now; 20M x 3 65 -> 47;
// 64M x 6 254 -> 227, 6.8 TB/s).  The loads of the next chunk are issued
// before the current one is reduced (two register buffers), so the memory
// stays busy while a wave computes.  Positions past a field's
// last whole vector load as NaN, which the finite test skips.  Every wave
// follows the same chunk sequence, so a change of field is
// workgroup-uniform: the running extrema are then folded into the field's
// keys.  The elements before a field's first 16-byte boundary and after its
// last whole vector (at most 3 + 3) are taken by workgroup 0, each lane
// with its own atomics.
template <int U>
__global__ __launch_bounds__(256) void field_range_kernel(RangeArgs a) {
    __shared__ int smin[4], smax[4];
    const uint64_t chunk = (uint64_t)U * 256;
    const uint64_t total = a.cpf * a.F;
    int mn = 0x7FFFFFFF, mx = (int)0x80000000;
    const uint64_t each = (total + gridDim.x - 1) / gridDim.x;
    uint64_t c = blockIdx.x * each;
    const uint64_t end = c + each < total ? c + each : total;
    if (c < end) {
        uint32_t cur = 0xFFFFFFFFu;
        RangeChunk r = range_chunk(a, c, chunk);
        f32x4 v[U];
        range_load<U>(r, chunk, v);
        for (;;) {
            const uint64_t cn = c + 1;
            RangeChunk rn = r;
            f32x4 w[U];
            if (cn < end) {
                rn = range_chunk(a, cn, chunk);
                range_load<U>(rn, chunk, w);
            }
            if (r.f != cur) {
                if (cur != 0xFFFFFFFFu) range_flush(a, cur, mn, mx, smin, smax);
                mn = 0x7FFFFFFF;
                mx = (int)0x80000000;
                cur = r.f;
            }
#pragma unroll
            for (int k = 0; k < U; k++) range_take4(v[k], mn, mx);
            if (cn >= end) break;
            c = cn;
            r = rn;
#pragma unroll
            for (int k = 0; k < U; k++) v[k] = w[k];
        }
        range_flush(a, cur, mn, mx, smin, smax);
    }
    if (blockIdx.x == 0) {
        // thread t < 8F: slot t % 8 of field t / 8 (slots 0-3 the head, 4-7 the tail)
        for (uint32_t t = threadIdx.x; t < 8u * a.F; t += 256) {
            const uint32_t f = t >> 3, j = t & 7u;
            const float* xf = a.x[f];
            const uint64_t head = ((16u - (reinterpret_cast<uintptr_t>(xf) & 15u)) & 15u) / 4u;
            const uint64_t h = head < a.n ? head : a.n;
            const uint64_t tail0 = h + 4 * ((a.n - h) / 4);
            const uint64_t i = j < 4 ? (uint64_t)j : tail0 + (j - 4);
            const bool live = j < 4 ? i < h : i < a.n;
            if (live && __builtin_isfinite(xf[i])) {
                const int k = order_key(xf[i]);
                atomicMin(&a.keys[f], k);
                atomicMax(&a.keys[a.F + f], k);
            }
        }
    }
}

}  // namespace

hipError_t launch_scan(const ScanArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(scan_lengths, dim3(1), dim3(kScanThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_copy(const CopyArgs& a, hipStream_t s) {
    if (a.nblocks == 0) return hipSuccess;
    if (a.copied) {
        const uint32_t rest = a.nblocks - a.placed * kSuper;
        hipLaunchKernelGGL(copy_rest, dim3(a.placed * kPlaceParts + (rest + kRestWaves - 1) / kRestWaves),
                           dim3(64 * kRestWaves), 0, s, a);
        return hipGetLastError();
    }
    const uint32_t groups = (a.nblocks + 3) / 4;
    if (a.left) hipLaunchKernelGGL(copy_records<true>, dim3(groups), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(copy_records<false>, dim3(groups), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_scan_batch(const ScanArgs* jobs, const BatchLaunch* L, const BatchShape& S,
                             hipStream_t s) {
    hipLaunchKernelGGL(scan_lengths_batch, dim3(S.scan_grid), dim3(kScanThreads), 0, s, jobs, L);
    return hipGetLastError();
}

hipError_t launch_copy_batch(const CopyArgs* jobs, const BatchLaunch* L, const BatchShape& S,
                             hipStream_t s) {
    if (S.grid)
        hipLaunchKernelGGL(copy_records_batch, dim3(S.copy_grid), dim3(256), 0, s, jobs, L);
    else
        hipLaunchKernelGGL(copy_records_batch_direct, dim3((S.direct_grid + 3) / 4), dim3(256), 0,
                           s, jobs, L);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t value, uint64_t count, hipStream_t s) {
    if (count == 0) return hipSuccess;
    uint64_t blocks = (count + 255) / 256;
    hipLaunchKernelGGL(fill_u32, dim3((uint32_t)blocks), dim3(256), 0, s, p, value, count);
    return hipGetLastError();
}

hipError_t launch_copy_words(uint32_t* dst, const uint32_t* src, uint32_t words, hipStream_t s) {
    hipLaunchKernelGGL(copy_words, dim3(1), dim3(256), 0, s, dst, src, words);
    return hipGetLastError();
}

hipError_t launch_reset_stats(uint32_t* zero, uint32_t nzero, int* keys, uint32_t nkeys,
                              hipStream_t s) {
    hipLaunchKernelGGL(reset_stats, dim3(1), dim3(256), 0, s, zero, nzero, keys, nkeys);
    return hipGetLastError();
}

hipError_t launch_stream_stats(const uint32_t* in, uint64_t in_words, uint64_t n, uint32_t F,
                               uint32_t B, unsigned long long* outliers, unsigned long long* raw,
                               uint32_t* err, hipStream_t s) {
    StatsArgs a{};
    a.in = in;
    a.in_words = in_words;
    a.n = n;
    a.F = F;
    a.B = B;
    a.nblocks = (uint32_t)nblocks_of(n, B);
    a.prefix = prefix_words(n, F, B);
    a.outliers = outliers;
    a.raw = raw;
    a.err = err;
    if (a.nblocks == 0) return hipSuccess;
    hipLaunchKernelGGL(stream_stats_kernel, dim3((a.nblocks + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_bound_check(const float* const* orig, const float* const* recon,
                              const uint32_t* perm, uint64_t n, uint32_t F, const float* eb,
                              unsigned long long* viol, unsigned long long* maxerr_bits,
                              double* sumsq, int* keys, hipStream_t s) {
    BoundArgs a{};
    for (uint32_t f = 0; f < F; f++) {
        a.orig[f] = orig[f];
        a.recon[f] = recon[f];
        a.eb[f] = eb[f];
    }
    a.perm = perm;
    a.n = n;
    a.F = F;
    a.viol = viol;
    a.maxerr_bits = maxerr_bits;
    a.sumsq = sumsq;
    a.keys = keys;
    const uint64_t need = ((n + kCheckChunk - 1) / kCheckChunk + kCheckWaves - 1) / kCheckWaves;
    const uint64_t most = (uint64_t)kCheckGroups * device_cu_count();
    const uint64_t groups = need < 1 ? 1 : (need < most ? need : most);
    if (sumsq)
        hipLaunchKernelGGL(bound_check_kernel<true>, dim3((uint32_t)groups), dim3(64 * kCheckWaves),
                           0, s, a);
    else
        hipLaunchKernelGGL(bound_check_kernel<false>, dim3((uint32_t)groups), dim3(64 * kCheckWaves),
                           0, s, a);
    return hipGetLastError();
}

namespace {

// The 2F range keys as floats in out[2F] (min, max per field): 0, 0 for a
// field with no finite value, a zero extreme as +0.0.
__global__ __launch_bounds__(64) void range_keys_to_floats(const int* __restrict__ keys, uint32_t F,
                                                           float* __restrict__ out) {
    for (uint32_t f = threadIdx.x; f < F; f += 64) {
        const int mn = keys[f], mx = keys[F + f];
        float lo = 0.0f, hi = 0.0f;
        if (mn <= mx) {
            lo = __int_as_float(mn ^ ((mn >> 31) & 0x7FFFFFFF));
            hi = __int_as_float(mx ^ ((mx >> 31) & 0x7FFFFFFF));
            if (lo == 0.0f) lo = 0.0f;
            if (hi == 0.0f) hi = 0.0f;
        }
        out[2 * f] = lo;
        out[2 * f + 1] = hi;
    }
}

}  // namespace

hipError_t launch_range_to_floats(const int* keys, uint32_t F, float* out, hipStream_t s) {
    hipLaunchKernelGGL(range_keys_to_floats, dim3(1), dim3(64), 0, s, keys, F, out);
    return hipGetLastError();
}

uint32_t device_cu_count() {
    constexpr int kDevices = 64;
    static std::atomic<int> cached[kDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return 256;
    int c = cached[dev].load(std::memory_order_relaxed);
    if (c <= 0) {
        if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            c <= 0)
            c = 256;
        cached[dev].store(c, std::memory_order_relaxed);
    }
    return (uint32_t)c;
}

hipError_t launch_field_range(const float* const* x, uint64_t n, uint32_t F, int* keys,
                              hipStream_t s) {
    // two workgroups per CU, eight 16-byte loads in flight per lane and buffer
    // (2 x 4 took 23, 50 and 238 us at the three sizes above, 4 x 4 26, 46 and
    // 228, 4 x 2 32, 55 and 230)
    constexpr int kLoads = 8;
    RangeArgs a{};
    for (uint32_t f = 0; f < F; f++) a.x[f] = x[f];
    a.n = n;
    a.F = F;
    a.keys = keys;
    const uint64_t chunk = (uint64_t)kLoads * 256;
    a.cpf = (n / 4 + chunk - 1) / chunk;
    if (a.cpf == 0) a.cpf = 1;  // workgroup 0 still takes the loose elements
    uint64_t groups = 2ull * device_cu_count();
    if (groups > a.cpf * F) groups = a.cpf * F;  // never more than the chunks
    hipLaunchKernelGGL(field_range_kernel<kLoads>, dim3((uint32_t)groups), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace gpz
