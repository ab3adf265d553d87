// Per-image selection (Algorithm 1 after the scores).  Images of at most
// kSmallSelectN tokens take select_small_kernel (one token per thread, both
// stages ranked in the same passes; described where it is defined).  Larger
// images take select_kernel: one 1024-thread workgroup per image, or several
// sharing the ranking of a large one.
//
// Keys are fp32 scores mapped to order-preserving u32 (-0 == +0).  Stage I
// keeps the K1 smallest Stage I keys (ties: lower index); Stage II orders
// X^rem by the Stage II key (ties: lower index) and keeps sorted positions
// 0, t, ..., (K2-1) t (or floor(j R / K2) in the real-interval variant); the
// output lists X^imp U X^div in token order.
//
// select_kernel keeps the image's keys in LDS.  One compute unit walks all
// of them, so its passes are bound by VALU issue (72 wavefront tiles on each
// SIMD for 18432 tokens) and are few: two over all tokens, then some over the
// tokens a workgroup ranks.
//
// Stage I looks for T, the K1-th smallest (key, index).  A round histograms the
// keys of a range into 1024 equal ranges of the order-preserving key and counts
// the keys below it; the next range is the one that holds T, so a round
// narrows it 512-fold or more whatever the values are.  The first range comes
// from 64 sampled keys around rank 64 K1 / N (a miss costs rounds over the side
// it names), and its histogram is taken as the keys arrive from memory.  At
// kMembers keys or fewer the range is left to the next pass; when one key value
// is left, the indices of its tokens are narrowed the same way (when all keys
// are equal, X^imp is the first K1 tokens).
//
// The second pass marks the keys below the range as X^imp, lists the range's
// members (ranked by counting: X^imp or not) and finds the workgroup's own
// tokens of X^rem: workgroup p of G on an image owns the tokens between samples
// p kSample / G and (p + 1) kSample / G of kSample sampled Stage II keys
// ((key, index) pairs where a sampled key repeats, so that equal keys are
// shared out too); G = 1 owns them all.  The tokens of X^rem below its own
// are counted, its own histogrammed into 1024 value buckets (bucket_of is
// non-decreasing in the key) and listed in bucket order, and a thread per listed
// token counts the members of its bucket smaller in (key, index) order.  Its
// rank in X^rem is the three counts' sum: exact, whatever the samples.  If
// many tokens share a bucket (kCountFixed) the own tokens are sorted instead, by
// a stable LSD radix sort of 16-bit indices (ordered compaction first, digits
// looked up by index, per-wavefront scatter offsets, passes over constant bytes
// skipped).
//
// In the output step every wavefront owns a contiguous, 64-aligned range of
// tokens; all results are exact and deterministic.
#include <type_traits>

#include "tr_internal.h"
#include "tr_wave.h"

namespace tr {
namespace {

constexpr int kThreads = 1024;
constexpr int kW = kThreads / kWave;
constexpr int kMaxSlots = 19;            // tokens per thread: images of at most 19456
constexpr int kUnr = 4;                  // tokens per thread a pass reads before it works on them
constexpr int kBuckets = kThreads;       // buckets of a histogram (one per thread in the scan)
constexpr uint32_t kMembers = 256;       // Stage I: list and rank the members of ranges this small
// Stage II: own tokens are ranked by counting while the squares of their buckets'
// sizes (the LDS reads) sum to at most kCountFixed + kCountPer for each of them.
// us of a selection of 16 images counted / sorted, by tokens and crowded buckets: 1500,
// one of 450 19.9 / 23.4, of 600 24.6 / 23.5; 2880, one of 600 26.1 / 33.7, of 1000 60.1
// / 33.9, four of 250 23.7 / 33.5, of 350 36.0 / 33.7; 4000, one of 600 27.6 / 41.0, of
// 1000 61.4 / 41.2, four of 250 33.7 / 41.0, of 450 52.8 / 41.2.
constexpr uint32_t kCountFixed = 100000, kCountPer = 120;
constexpr int kSample = 128;             // Stage II: samples that share out an image
constexpr int kShareRem = 4096;          // Stage II: share images with this many remaining tokens
constexpr int kListN = 2 * kShareRem;    // images below this have LDS for every token as a pair
constexpr int kMaxSplitGroups = 64;      // most workgroups sharing the ranking of one large image
static_assert((uint32_t)(kListN / 2) * (kListN / 2) > kCountFixed + kCountPer * kMaxSlots * kThreads,
              "a bucket that the list cannot hold is sorted");
static_assert(kMembers <= (uint32_t)kThreads, "one thread per listed Stage I member");
static_assert((kMaxSplitGroups & (kMaxSplitGroups - 1)) == 0 && kMaxSplitGroups * 2 <= kSample,
              "two samples or more to a workgroup");
static_assert(kShareRem >= 4 * kSample, "samples of a shared image are distinct tokens");
static_assert(kMaxSlots <= 32 && kMaxSlots * kThreads <= 65535, "16-bit indices, and products of ranks below 2^32");

// ---- LDS layout (same arithmetic on host and device) -----------------------
struct LdsLayout {
    size_t ks, ki, bimp, bsel, area, slots, misc, list, list_bytes, total;
};

__host__ __device__ inline size_t align_up(size_t v, size_t a) { return (v + a - 1) & ~(a - 1); }

// Without Stage II (no image of the launch has K2 > 0) there is no ks and no list.
//   ks    u32[n]        Stage II keys by token index
//   ki    u32[n]        Stage I keys; once X^imp is known the list of the own
//                       tokens (below), or the two u16[n] index buffers of the
//                       radix sort
//   bimp  u32[nw]       X^imp bitmap (nw = 2 ceil(n / 64)); the radix sort of a
//                       shared image: the tokens it leaves out
//   bsel  u32[nw]       X^imp U X^div bitmap
//   area  u32[2048]     16-byte aligned: [0, 1024) histogram, [1024, 2048) by
//                       phase the samples (kS*), Stage I's
//                       members u64[kMembers], Stage II's bucket cursors; or
//                       u16[256][W] digit counts / offsets of the radix sort
//   slots u32[8][W]     per-wavefront partial values, one row per use
//   misc  u32[16]       broadcast words (kM*)
//   list  list_bytes    the own tokens in bucket order, u64 (key << 32 | index).
//                       n < kListN: a region of u64[n], else the bytes of ki
//                       (a share of a large image is far smaller; an image that
//                       one workgroup ranks alone is listed in parts)
__host__ __device__ inline LdsLayout lds_layout(int n, bool two = true)
{
    LdsLayout L;
    const size_t nw = 2 * (((size_t)n + 63) / 64);
    size_t o = 0;
    L.ks = o;
    if (two) o += 4 * (size_t)n;
    L.ki = o;
    o += 4 * (size_t)n;
    L.bimp = o;
    o += 4 * nw;
    L.bsel = o;
    o += 4 * nw;
    o = align_up(o, 16);
    L.area = o;
    o += 4 * 2 * kBuckets;
    L.slots = o;
    o += 4 * 8 * kW;
    L.misc = o;
    o += 4 * 16;
    if (n < kListN) {
        L.list = o;
        L.list_bytes = two ? 8 * (size_t)n : 0;
        o += L.list_bytes;
    } else {
        L.list = align_up(L.ki, 8);
        L.list_bytes = 4 * (size_t)n - (L.list - L.ki);
    }
    L.total = o;
    return L;
}

// LDS a launch needs for images of at most nmax tokens: the largest layout of
// any n <= nmax (it is not monotonic at kListN).
__host__ __device__ inline size_t launch_lds(int nmax, bool two = true)
{
    const size_t big = lds_layout(nmax, two).total;
    if (nmax < kListN || !two) return big;
    const size_t small = lds_layout(kListN - 1).total;
    return big > small ? big : small;
}

// Words of area + 1024 while samples are ranked.
constexpr int kSRows = 0;      // u64[2][64]: the two kinds' 64 samples
constexpr int kSRanks = 256;   // u16[8][kSample]: partial ranks
constexpr int kSSorted = 256 + 4 * kSample;   // u32[kSample]: sampled Stage II keys in order
static_assert(kSSorted >= 2 * (int)kMembers && kSSorted + kSample <= kBuckets, "above Stage I's members, in the area");

// Words of misc.
constexpr int kMBracket = 0;   // Stage I's sampled range (2 keys)
constexpr int kMQuant = 2;     // Stage II's value range (2 keys)
constexpr int kMRound = 4;     // a round's bucket, the rank inside it, its size
constexpr int kMCount = 7;     // listed members
constexpr int kMOwn = 8;       // first pair owned, first pair not owned any more (2 u64)

// ---- helpers -------------------------------------------------------------------
// IEEE order -> unsigned order; -0 and +0 map to the same key.
__device__ __forceinline__ uint32_t order_key(float f)
{
    const uint32_t u = __float_as_uint(f + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Inverse of order_key.
__device__ __forceinline__ float key_value(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k ^ 0x80000000u) : ~k);
}

__device__ __forceinline__ uint64_t pair_of(uint32_t key, uint32_t i) { return ((uint64_t)key << 32) | i; }

__device__ __forceinline__ uint64_t lanes_below(int lane) { return (1ull << lane) - 1ull; }

// Mask of active lanes whose 8-bit digit equals this lane's digit.
__device__ __forceinline__ uint64_t same_digit(uint32_t digit, bool active)
{
    uint64_t m = __ballot(active);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const bool bit = (digit >> b) & 1u;
        const uint64_t set = __ballot(active && bit);
        m &= bit ? set : ~set;
    }
    return m;
}

__device__ __forceinline__ bool is_leader(uint64_t m, int lane)
{
    return m && (int)(__ffsll((long long)m) - 1) == lane;
}

__device__ __forceinline__ bool bit_of(const uint32_t* bm, int i) { return (bm[i >> 5] >> (i & 31)) & 1u; }

// A wavefront writes the 64-bit ballot of tile `base` into the tile's two
// bitmap words (base is a multiple of 64 and every bitmap starts 8-byte
// aligned, so the pair is one aligned 64-bit store).
__device__ __forceinline__ void put_tile_bits(uint32_t* bm, int base, uint64_t bits, int lane)
{
    if (lane == 0) *reinterpret_cast<uint64_t*>(bm + (base >> 5)) = bits;
}

// Contiguous 64-aligned token range of wavefront w.
__device__ __forceinline__ void wave_range(int n, int w, int& beg, int& end)
{
    const int seg = (((n + kW - 1) / kW) + 63) & ~63;
    beg = w * seg < n ? w * seg : n;
    end = beg + seg < n ? beg + seg : n;
}

// Cross-wavefront reductions of one LDS row of per-wavefront values: lane l
// reads entry l, the wavefront reduces in registers.
static_assert(kW <= kWave, "one row entry per lane");

// Sum of the entries of wavefronts 0 .. w-1.
__device__ __forceinline__ uint32_t sum_before(const uint32_t* row, int w, int lane)
{
    return wave_sum_u32(lane < w ? row[lane] : 0u);
}

__device__ __forceinline__ uint32_t max_all(const uint32_t* row, int lane)
{
    return wave_max_u32(lane < kW ? row[lane] : 0u);
}

// Exclusive prefix over wavefronts of a per-wavefront count.
__device__ __forceinline__ uint32_t wave_prefix(uint32_t count, uint32_t* row)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    if (lane == 0) row[w] = count;
    __syncthreads();
    return sum_before(row, w, lane);
}

struct Img {
    int row_off, n, k1, k2, t, out_off;
};

__device__ __forceinline__ Img image_of(const SelectArgs& a, int local)
{
    ImageDesc d;
    if (a.uniform) {
        d = a.desc[0];
        const int img = a.img0 + local;
        d.row_off = img * d.n;
        d.out_off = img * (d.k1 + d.k2);
    } else {
        d = a.desc[local];
    }
    return Img{d.row_off, d.n, d.k1, d.k2, d.t, d.out_off};
}

// X^div positions in the ascending order of X^rem (R tokens, K2 picks).
// Algorithm 1: 0, t, ..., (K2 - 1) t.  Real-interval variant (the interval
// R / K2 of the method's prose): floor(j R / K2), j < K2.  Every product
// stays below 2^32 because R, K2 <= 65535.
struct Stride {
    uint32_t t, R, K2;
    bool real;
    // Is rank r a pick?  Real variant: the smallest j with floor(j R / K2) >=
    // r is ceil(r K2 / R); r is a pick iff that j is in range and lands on r.
    __device__ __forceinline__ bool picks(uint32_t r) const
    {
        if (!real) return r % t == 0 && r < K2 * t;
        const uint32_t j = (r * K2 + R - 1) / R;
        return j < K2 && (j * R) / K2 == r;
    }
    __device__ __forceinline__ uint32_t pos(uint32_t j) const { return real ? (j * R) / K2 : j * t; }
};

// Bucketing of one key over [lo, hi] (order keys) into nb buckets.
struct Bucketing {
    int32_t mode;      // 0: value buckets; 1: order-key buckets; 2: every key equal
    float fmin, scale;
    uint32_t kmin;
    int32_t shift;
};

// kmin / kmax: the true range of the keys (order keys); value buckets need
// every key to be a number (NaN keys lie outside [-inf, +inf] in key order).
__device__ __forceinline__ Bucketing make_bucketing(uint32_t lo, uint32_t hi, uint32_t kmin, uint32_t kmax, int nb)
{
    Bucketing b;
    b.mode = 2;
    b.kmin = lo;
    b.fmin = key_value(lo);
    b.scale = 0.f;
    b.shift = 0;
    if (kmin == kmax) return b;
    const bool no_nan = kmin >= 0x007fffffu && kmax <= 0xff800000u;
    const float width = key_value(hi) - b.fmin;
    const float scale = (float)nb / width;
    if (no_nan && width > 0.f && width < 3.0e38f && scale < 3.0e38f) {
        b.mode = 0;
        b.scale = scale;
        return b;
    }
    b.mode = 1;
    const uint32_t span = hi - lo;
    int sh = 0;
    while (sh < 31 && (span >> sh) >= (uint32_t)nb) ++sh;
    b.shift = sh;
    return b;
}

// Non-decreasing in the key; always in [0, nb).
__device__ __forceinline__ int bucket_of(const Bucketing& b, uint32_t k, int nb)
{
    if (b.mode == 0) {
        const float x = (key_value(k) - b.fmin) * b.scale;   // NaN only if a key is NaN (then mode 1)
        return x <= 0.f ? 0 : (x >= (float)(nb - 1) ? nb - 1 : (int)x);
    }
    if (b.mode == 1) {
        if (k <= b.kmin) return 0;
        const uint32_t q = (k - b.kmin) >> b.shift;
        return q >= (uint32_t)nb ? nb - 1 : (int)q;
    }
    return 0;
}

// The keys of ranks lo_rank and hi_rank among 64 sampled keys of an image (all
// of them for N <= 64; a rank outside [0, 64) publishes nothing), by one
// wavefront without the workgroup:
// lane k loads sample k (token floor(k N / 64)), the wave stages the samples
// as distinct (key << 6 | k) values in its own LDS row, every lane ranks its
// sample among the 64 (two per 16-byte broadcast read), and the lanes holding
// ranks lo_rank and hi_rank publish their keys in out[0], out[1].
__device__ __forceinline__ int sample_index(int N, int lane)
{
    return N > kWave ? (int)(((int64_t)lane * N) >> 6) : lane;
}

template <int Q = 16>   // pairs of samples in flight
__device__ __forceinline__ void sample_quantiles(uint32_t key, int lane, uint64_t* samp, int lo_rank, int hi_rank,
                                                 uint32_t* out)
{
    const uint64_t mine = ((uint64_t)key << 6) | (uint64_t)lane;
    samp[lane] = mine;
    // LDS operations of one wavefront complete in order: the row written
    // above is visible to the reads below
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const ulonglong2* sv = reinterpret_cast<const ulonglong2*>(samp);
    int r = 0;
#pragma unroll
    for (int h = 0; h < 32 / Q; ++h) {
        ulonglong2 q[Q];
#pragma unroll
        for (int j = 0; j < Q; ++j) q[j] = sv[Q * h + j];
#pragma unroll
        for (int j = 0; j < Q; ++j) r += (q[j].x < mine ? 1 : 0) + (q[j].y < mine ? 1 : 0);
    }
    if (r == lo_rank) out[0] = (uint32_t)(mine >> 6);
    if (r == hi_rank) out[1] = (uint32_t)(mine >> 6);
}

// Exact rank of `me` = (key << 32 | index) among the n > 1 members
// list[beg, beg + n) of its bucket, plus beg (the tokens of lower buckets).
__device__ __forceinline__ uint32_t rank_in(const uint64_t* list, uint32_t beg, uint32_t n, uint64_t me)
{
    const uint32_t end = beg + n;
    uint32_t r = beg, j = beg;
    for (; j + 4 <= end; j += 4) {
        const uint64_t m0 = list[j], m1 = list[j + 1], m2 = list[j + 2], m3 = list[j + 3];
        r += (m0 < me) + (m1 < me) + (m2 < me) + (m3 < me);
    }
    for (; j < end; ++j) r += list[j] < me ? 1u : 0u;
    return r;
}

// Lane t's value of a 64-bit register, on every lane (t wavefront-uniform).
__device__ __forceinline__ uint64_t lane_u64(uint64_t v, int t)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, t);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), t);
    return ((uint64_t)hi << 32) | lo;
}

// The tokens not in `skip` (R of them) in (key, index) order: ordered compaction,
// then a stable LSD radix sort of 16-bit indices over the bytes that `vary`
// says can differ.  Returns the sorted list, one of idx_a / idx_b (n u16
// each); the workgroup is past a barrier.
__device__ __forceinline__ const uint16_t* radix_sort(const uint32_t* ks, const uint32_t* skip, int N, int R, uint32_t vary,
                                      uint16_t* idx_a, uint16_t* idx_b, uint16_t* hist, uint32_t* row_c,
                                      uint32_t* row_s)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    int beg, end;
    wave_range(N, w, beg, end);
    uint32_t rc = 0;
    for (int base = beg; base < end; base += kWave) {
        const int i = base + lane;
        rc += __popcll(__ballot(i < end && !bit_of(skip, i)));
    }
    uint32_t pos = wave_prefix(rc, row_c);
    for (int base = beg; base < end; base += kWave) {
        const int i = base + lane;
        const bool keep = i < end && !bit_of(skip, i);
        const uint64_t bk = __ballot(keep);
        if (keep) idx_a[pos + __popcll(bk & lanes_below(lane))] = (uint16_t)i;
        pos += (uint32_t)__popcll(bk);
    }
    int begR, endR;
    wave_range(R, w, begR, endR);
    uint16_t* src = idx_a;
    uint16_t* dst = idx_b;
    for (int shift = 0; shift < 32; shift += 8) {
        if (((vary >> shift) & 255u) == 0) continue;   // every key has the same byte here
        uint32_t* h32 = reinterpret_cast<uint32_t*>(hist);
        for (int i = tid; i < 128 * kW; i += kThreads) h32[i] = 0;
        __syncthreads();
        for (int base = begR; base < endR; base += kWave) {
            const int i = base + lane;
            const bool act = i < endR;
            const uint32_t id = act ? src[i] : 0u;
            const uint32_t dg = act ? (ks[id] >> shift) & 255u : 0u;
            const uint64_t m = same_digit(dg, act);
            if (act && is_leader(m, lane)) hist[dg * kW + w] = (uint16_t)(hist[dg * kW + w] + __popcll(m));
        }
        __syncthreads();
        {   // exclusive scan of hist in (digit, wavefront) order, 4 entries per thread
            const int e = tid * 4;
            const uint2 hv = *reinterpret_cast<const uint2*>(hist + e);
            const uint32_t h0 = hv.x & 0xffffu, h1 = hv.x >> 16, h2 = hv.y & 0xffffu, h3 = hv.y >> 16;
            const uint32_t v = h0 + h1 + h2 + h3;
            const uint32_t inc = wave_scan_add(v);
            if (lane == kWave - 1) row_s[w] = inc;
            __syncthreads();
            const uint32_t b0 = inc - v + sum_before(row_s, w, lane);
            const uint32_t o1 = b0 + h0, o2 = o1 + h1, o3 = o2 + h2;
            *reinterpret_cast<uint2*>(hist + e) = make_uint2(b0 | (o1 << 16), o2 | (o3 << 16));
        }
        __syncthreads();
        for (int base = begR; base < endR; base += kWave) {
            const int i = base + lane;
            const bool act = i < endR;
            const uint32_t id = act ? src[i] : 0u;
            const uint32_t dg = act ? (ks[id] >> shift) & 255u : 0u;
            const uint64_t m = same_digit(dg, act);
            const uint32_t off = act ? hist[dg * kW + w] : 0u;
            if (act) dst[off + __popcll(m & lanes_below(lane))] = (uint16_t)id;
            if (act && is_leader(m, lane)) hist[dg * kW + w] = (uint16_t)(off + __popcll(m));
        }
        __syncthreads();
        uint16_t* tmp = src;
        src = dst;
        dst = tmp;
    }
    __syncthreads();   // the compaction (or the last pass) is visible to every reader
    return src;
}

// Word of an image's bitmaps at which this lane's tile of the output step starts,
// or -1 for a lane without a tile.
__device__ __forceinline__ int tile_word(int n)
{
    int beg, end;
    wave_range(n, (int)threadIdx.x / kWave, beg, end);
    const int at = beg + kWave * ((int)threadIdx.x & (kWave - 1));
    return at < end ? at >> 5 : -1;
}

// X* in ascending token index: out_idx (image-local), out_src, out_rows.
// Lane t of each wavefront holds the 64-bit words of X* (sel) and X^imp (imp) of
// the wavefront's t-th tile (a range has at most 64 tiles at the capacity's N;
// tile_word says where a lane's words start).
__device__ __forceinline__ void emit(const SelectArgs& a, const Img& d, uint64_t sel, uint64_t imp, uint32_t* row)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    int beg, end;
    wave_range(d.n, w, beg, end);
    const int tiles = (end - beg + kWave - 1) / kWave;
    const int valid = end - (beg + kWave * lane);   // tokens of this lane's tile inside the image
    if (valid < kWave) sel &= valid > 0 ? (1ull << valid) - 1ull : 0ull;
    uint32_t opos = wave_prefix(wave_sum_u32((uint32_t)__popcll(sel)), row);
    const int K = d.k1 + d.k2;
    for (int t = 0; t < tiles; ++t) {
        const uint64_t m = lane_u64(sel, t), im = lane_u64(imp, t);
        const int i = beg + kWave * t + lane;
        const int slot = (int)opos + __popcll(m & lanes_below(lane));
        if (((m >> lane) & 1ull) && slot < K) {   // never more than K writes, whatever the keys
            const int o = d.out_off + slot;
            a.out_idx[o] = i;
            if (a.out_src) a.out_src[o] = ((im >> lane) & 1ull) ? 0 : 1;
            if (a.out_rows) a.out_rows[o] = d.row_off + i;
        }
        opos += (uint32_t)__popcll(m);
    }
}

// One pass over the image: f(tokens of this thread) for kUnr tokens at a time,
// i[v] = (u + v) kThreads + threadIdx.x, slot u + v.  Whole wavefronts take
// part; indices beyond the image come too (f masks them), their reads clamped.
template <typename F>
__device__ __forceinline__ void for_tokens(int N, F f)
{
    for (int u = 0; u * kThreads < N; u += kUnr) f(u, u * kThreads + (int)threadIdx.x);
}

__device__ __forceinline__ void read_keys(const uint32_t* v, int i0, int N, uint32_t (&out)[kUnr])
{
#pragma unroll
    for (int q = 0; q < kUnr; ++q) out[q] = v[min(i0 + q * kThreads, N - 1)];
}

// A barrier for what is exchanged through LDS: loads from memory stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Append (key, index) of the lanes of `bm` (not empty) to `list`, reserving the
// wavefront's slots with one atomic on the counter `cnt`.
__device__ __forceinline__ void append_member(uint64_t bm, uint32_t key, int i, uint64_t* list, uint32_t* cnt,
                                              int lane)
{
    uint32_t b0 = 0;
    if (lane == 0) b0 = atomicAdd(cnt, (uint32_t)__popcll(bm));
    b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b0);
    const uint32_t at = b0 + (uint32_t)__popcll(bm & lanes_below(lane));
    if ((bm >> lane & 1ull) && at < kMembers) list[at] = pair_of(key, (uint32_t)i);   // never beyond, whatever the keys
}

// The scan after one histogram of Stage I: thread t owns bucket t of H (zero on
// return); below / inside: the tokens below the range / in it.  The bucket that
// holds the K1-th smallest goes to misc[kMRound ..].
__device__ __forceinline__ void stage1_scan(uint32_t wave_below, uint32_t K1, uint32_t* H, uint32_t* misc,
                                            uint32_t* row_b, uint32_t* row_c, uint32_t& below, uint32_t& inside)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    if (lane == 0) row_b[w] = wave_below;
    __syncthreads();
    const uint32_t c = H[tid];
    H[tid] = 0u;
    const uint32_t inc = wave_scan_add(c);
    if (lane == kWave - 1) row_c[w] = inc;
    __syncthreads();
    below = sum_before(row_b, kW, lane);
    inside = sum_before(row_c, kW, lane);
    const uint32_t start = below + inc - c + sum_before(row_c, w, lane);
    if (start < K1 && K1 <= start + c) {
        misc[kMRound] = (uint32_t)tid;
        misc[kMRound + 1] = K1 - start;
        misc[kMRound + 2] = c;
    }
    __syncthreads();
}

// One round's histogram over the keys in LDS: tokens with lo <= v <= hi go to
// bucket (v - lo) >> sh, those below lo are counted for the wavefront.  v is
// the key, or (INDEX) the index of the tokens whose key is `only`, all of them in
// buckets of 32.  Atomics of many lanes on one bucket run one after the other
// (3600 tokens of one key: 3 us), so a range of one key is counted by ballots.
constexpr int kIdxShift = 5;

template <bool INDEX>
__device__ uint32_t stage1_histogram(const uint32_t* ki, int N, uint32_t only, uint32_t lo, uint32_t hi, int sh,
                                     uint32_t* H)
{
    const int lane = threadIdx.x & (kWave - 1);
    uint32_t nb = 0, one = 0;
    for_tokens(N, [&](int, int i0) {
        uint32_t k[kUnr];
        read_keys(ki, i0, N, k);
#pragma unroll
        for (int q = 0; q < kUnr; ++q) {
            const int i = i0 + q * kThreads;
            const uint32_t v = INDEX ? (uint32_t)i : k[q];
            const bool have = i < N && (!INDEX || k[q] == only);
            if constexpr (INDEX) {   // a tile's tokens fall into two buckets: lanes 0 and 32 count them
                static_assert(kIdxShift == 5, "half a tile to a bucket");
                const uint64_t m = __ballot(have);
                const uint32_t n = lane < 32 ? (uint32_t)__popc((uint32_t)m) : (uint32_t)__popc((uint32_t)(m >> 32));
                if ((lane & 31) == 0 && n) atomicAdd(&H[v >> kIdxShift], n);
            } else {
                const bool in = have && v - lo <= hi - lo;
                nb += (uint32_t)__popcll(__ballot(have && v < lo));
                if (lo == hi) one += (uint32_t)__popcll(__ballot(in));
                else if (in) atomicAdd(&H[(v - lo) >> sh], 1u);
            }
        }
    });
    if (!INDEX && lane == 0 && one) atomicAdd(&H[0], one);
    return nb;
}

// Bits to drop so that the range [lo, hi] fits the buckets.
__device__ __forceinline__ int range_shift(uint32_t lo, uint32_t hi)
{
    const int bits = hi > lo ? 32 - __clz((int)(hi - lo)) : 0;
    static_assert(kBuckets == 1 << 10, "ten bits of a range");
    return bits > 10 ? bits - 10 : 0;
}

// The tokens that hold T: (lo, ilo) <= (key, index) <= (hi, ihi), at most
// kMembers of them, T the need-th smallest.
struct Boundary {
    uint32_t lo, hi, ilo, ihi, need;
    bool tie;   // one key value, narrowed by index
};

// From the first range's scan on.
__device__ __forceinline__ Boundary stage1_boundary(const uint32_t* ki, int N, uint32_t K1, uint32_t lo, uint32_t hi,
                                                    uint32_t below, uint32_t inside, uint32_t* H, uint32_t* misc,
                                                    uint32_t* row_b, uint32_t* row_c)
{
    Boundary r;
    uint32_t m;
    for (;;) {
        if (K1 <= below) {   // the sampled range lies above T
            hi = lo - 1;
            lo = 0u;
        } else if (K1 > below + inside) {   // or below it
            lo = hi + 1;
            hi = 0xffffffffu;
        } else {
            const int sh = range_shift(lo, hi);
            r.need = misc[kMRound + 1];
            m = misc[kMRound + 2];
            lo += misc[kMRound] << sh;
            hi = min(hi - lo, (1u << sh) - 1u) + lo;
            if (m <= kMembers || sh == 0) break;
        }
        const uint32_t nb = stage1_histogram<false>(ki, N, 0u, lo, hi, range_shift(lo, hi), H);
        stage1_scan(nb, K1, H, misc, row_b, row_c, below, inside);
    }
    r.lo = lo;
    r.hi = hi;
    r.ilo = 0u;
    r.ihi = 0xffffffffu;
    r.tie = m > kMembers;
    if (r.tie && m == (uint32_t)N) {   // every key is equal: the first K1 tokens, no boundary left
        r.need = 0u;
        r.ilo = K1;
        r.ihi = K1 - 1u;
    } else if (r.tie) {   // tokens of one key value: those of the lowest indices
        static_assert(kMaxSlots * kThreads <= kBuckets << kIdxShift, "every index has a bucket");
        const uint32_t nb = stage1_histogram<true>(ki, N, lo, 0u, (uint32_t)N - 1u, kIdxShift, H);
        stage1_scan(nb, r.need, H, misc, row_b, row_c, below, inside);
        r.need = misc[kMRound + 1];
        r.ilo = misc[kMRound] << kIdxShift;
        r.ihi = r.ilo + ((1u << kIdxShift) - 1u);
    }
    return r;
}

// What the second pass needs of the workgroup's share of X^rem.
struct Share {
    uint64_t lo, hi;   // first pair owned, first pair not owned any more
    bool open;         // no upper end
};

// The second pass: X^imp bits (bimp, and bsel if given; null: none), the
// boundary's members, the own tokens (bit u of `own`: slot u) and the count
// of X^rem below them for the wavefront.  EXACT compares (key, index); without
// it the boundary and the share are ranges of keys.  The counts come from
// ballots of single comparisons, combined as scalars: a ballot of a combined
// condition costs two vector instructions more, and a tile has about ten.
template <bool EXACT, bool TWO, bool FULL>   // FULL: every token read is one of the image
__device__ __forceinline__ void second_pass_step(const uint32_t* ki, const uint32_t* ks, int N, int u, const Boundary& bd,
                                                 uint64_t imp_end, bool members_left, const Share& sh,
                                                 uint64_t* members, uint32_t* count, uint32_t* bimp, uint32_t* bsel,
                                                 uint32_t& own, uint32_t& rem_below)
{
    const int lane = threadIdx.x & (kWave - 1), i0 = u * kThreads + (int)threadIdx.x;
    const uint64_t mhi = pair_of(bd.hi, bd.ihi);
    const uint32_t klo = (uint32_t)(sh.lo >> 32), khi = sh.open ? 0xffffffffu : (uint32_t)(sh.hi >> 32) - 1u;
    uint32_t qi[kUnr], qs[kUnr] = {};
    if constexpr (FULL) {
#pragma unroll
        for (int q = 0; q < kUnr; ++q) {
            qi[q] = ki[i0 + q * kThreads];
            if constexpr (TWO) qs[q] = ks[i0 + q * kThreads];
        }
    } else {
        read_keys(ki, i0, N, qi);
        if constexpr (TWO) read_keys(ks, i0, N, qs);
    }
#pragma unroll
    for (int q = 0; q < kUnr; ++q) {
        const int i = i0 + q * kThreads, tb = i - lane;
        const bool valid = FULL || i < N;
        const uint64_t pi = pair_of(qi[q], (uint32_t)i), ps = pair_of(qs[q], (uint32_t)i);
        const bool imp = EXACT ? pi < imp_end : qi[q] < bd.lo;
        const bool upto = EXACT ? pi <= mhi : qi[q] < bd.hi + 1u;   // X^imp or a member
        const bool below = EXACT ? ps < sh.lo : qs[q] < klo;
        const bool under = EXACT ? sh.open || ps < sh.hi : qs[q] <= khi;
        const uint64_t vm = FULL ? ~0ull : __ballot(valid);
        const uint64_t mi = __ballot(imp) & vm;
        const uint64_t mm = EXACT && !members_left ? 0ull : __ballot(upto) & vm & ~mi;
        if constexpr (TWO) rem_below += (uint32_t)__popcll(__ballot(below) & vm & ~(mi | mm));
        if (mm) append_member(mm, qi[q], i, members, count, lane);
        if (bimp && (FULL || tb < N)) {
            put_tile_bits(bimp, tb, mi, lane);
            if (bsel) put_tile_bits(bsel, tb, mi, lane);
        }
        const bool rem = valid && !(EXACT ? imp || (members_left && upto) : upto);   // imp implies upto
        if constexpr (TWO) own |= rem && !below && under ? 1u << (u + q) : 0u;
    }
}

template <bool EXACT, bool TWO>
__device__ __forceinline__ void second_pass(const uint32_t* ki, const uint32_t* ks, int N, const Boundary& bd,
                                            uint64_t imp_end, bool members_left, const Share& sh, uint64_t* members,
                                            uint32_t* count, uint32_t* bimp, uint32_t* bsel, uint32_t& own,
                                            uint32_t& rem_below)
{
    int u = 0;
    if constexpr (!EXACT)
        for (; (u + kUnr) * kThreads <= N; u += kUnr)
            second_pass_step<false, TWO, true>(ki, ks, N, u, bd, imp_end, members_left, sh, members, count, bimp,
                                                bsel, own, rem_below);
    for (; u * kThreads < N; u += kUnr)
        second_pass_step<EXACT, TWO, false>(ki, ks, N, u, bd, imp_end, members_left, sh, members, count, bimp, bsel,
                                             own, rem_below);
}

// A place in [0, n), n < 65536, that differs from k to k.
__device__ __forceinline__ uint32_t scatter(int k, uint32_t n)
{
    return (((uint32_t)k * 2654435761u) >> 16) * n >> 16;
}

// Sample k of a shared image: one token of the k-th of kSample equal parts,
// at a place that differs from part to part, so that a period in the tokens
// (frames of a clip) does not meet a period in the samples.
__device__ __forceinline__ int sample_token(int k, int N)
{
    return (int)((uint32_t)k * (uint32_t)N / kSample + scatter(k, (uint32_t)N / kSample));
}

// The keys are loaded in one burst, S of each kind a thread (N <= S kThreads);
// the samples, loaded before them, are ranked while they arrive.
// S is 4, 10 or 19 by the launch's largest image: a thread loads S keys of each
// kind whatever its image, clamped reads beyond it.
//
// Bound by the latency of its phases (a dozen barriers of sixteen wavefronts, a
// round trip to memory) and by VALU issue in the two passes over all tokens.
// A workgroup of the 4 x 18432 clips, us from its start, against a kernel that
// bucketed every key from LDS and all of X^rem in every workgroup: samples ranked
// 2.9, keys and first histogram 6.9 (6.6), boundary 9.1 (12), second pass 13-14
// (16), own tokens' histogram and scan 15-16 (20), ranked 16-18 (23).  Selection
// alone of 24 images of up to 18000 tokens: 39 -> 28 us.  Tried and left out: the
// keys in registers instead of LDS (19 + 19 a thread, every pass unrolled over
// them: 10000 instructions, not run); comparisons of (key, index) pairs in every
// pass (second pass 1.2 us more); value buckets over sampled quantiles with the
// tails clamped into the end buckets (a tail of 3 % of 18000 tokens went to the
// radix sort: 56 us).
//
// Without TWO no image of the launch has a Stage II (K1 = K, as at lambda = 1):
// nothing of its keys is loaded, kept or ranked.
template <int S, bool TWO>
__global__ __launch_bounds__(kThreads) void select_kernel(SelectArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int G = TWO && a.groups > 0 ? a.groups : 1;
    const int local = (int)blockIdx.x / G, part = (int)blockIdx.x % G;
    const int img = a.img0 + local;
    const Img d = image_of(a, local);
    const int N = d.n, K1 = d.k1, K2 = TWO ? d.k2 : 0, R = N - K1;
    const bool split = TWO && G > 1 && K2 > 0 && R >= kShareRem;   // as select_shares
    if (part > 0 && !split) return;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const LdsLayout L = lds_layout(N, TWO);
    uint32_t* ks = reinterpret_cast<uint32_t*>(smem + L.ks);
    uint32_t* ki = reinterpret_cast<uint32_t*>(smem + L.ki);
    uint32_t* bimp = reinterpret_cast<uint32_t*>(smem + L.bimp);
    uint32_t* bsel = reinterpret_cast<uint32_t*>(smem + L.bsel);
    uint32_t* H = reinterpret_cast<uint32_t*>(smem + L.area);
    uint32_t* cur = H + kBuckets;
    uint32_t* slots = reinterpret_cast<uint32_t*>(smem + L.slots);
    uint32_t* misc = reinterpret_cast<uint32_t*>(smem + L.misc);
    uint64_t* own64 = reinterpret_cast<uint64_t*>(misc + kMOwn);
    const float* fi = a.key_imp + d.row_off;
    const float* fs = a.key_s + d.row_off;

    // ---- keys, samples, ranges -------------------------------------------------
    const float* fq = !TWO || w == 0 ? fi : fs;   // 64 samples of either kind, ranked by wavefronts 0 and 1
    const int iq = sample_index(N, lane) + (N > kWave ? (int)scatter(lane, (uint32_t)N / kWave) : 0);
    const float vq = fq[min(iq, N - 1)];
    int ia = 0, ib = 0;   // one block of the shared image's samples, and one it is compared with
    if (split) {
        ia = sample_token((w & 1) * kWave + lane, N);
        ib = sample_token((w >> 1 & 1) * kWave + lane, N);
    }
    const float va = TWO ? fs[ia] : 0.f, vb = TWO ? fs[ib] : 0.f;
    __builtin_amdgcn_sched_barrier(0);   // the samples' loads leave first
    float vi[S], vs[S];
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const uint32_t at = 4u * (uint32_t)min(u * kThreads + tid, N - 1);   // 32 bits: base + offset loads
        vi[u] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(fi) + at);
        if constexpr (TWO) vs[u] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(fs) + at);
    }
    __builtin_amdgcn_sched_barrier(0);
    H[tid] = 0u;
    if (tid == 0) misc[kMCount] = 0u;
    // Stage I's first range: the samples about three standard deviations to
    // either side of rank 64 K1 / N; past the ends, three times as far as it is
    // wide (one image in ten missed T with 2.5 and once: 2 to 4 us each)
    const float at = (float)kWave * (float)K1 / (float)N;
    const float off = 3.0f * sqrtf(at * fmaxf((float)kWave - at, 0.f) / (float)kWave) + 3.0f;
    const int last = min(N, kWave) - 1;
    const int rlo = (int)floorf(at - off), rhi = (int)ceilf(at + off);
    const uint32_t qkey = iq < N ? order_key(vq) : 0xffffffffu;
    uint64_t* rows = reinterpret_cast<uint64_t*>(cur + kSRows);
    uint16_t* ranks = reinterpret_cast<uint16_t*>(cur + kSRanks);
    uint32_t* sorted_keys = cur + kSSorted;
    if (w == 0)
        sample_quantiles<8>(qkey, lane, rows, N > kWave ? max(rlo, 0) : 0, N > kWave ? min(rhi, last) : last,
                            &misc[kMBracket]);
    if (TWO && w == 1 && !split)
        sample_quantiles<8>(qkey, lane, rows + kWave, N > kWave ? 1 : 0, N > kWave ? kWave - 2 : last, &misc[kMQuant]);
    const uint64_t smine = pair_of(order_key(va), (uint32_t)ia);
    if (split) {   // a quarter of the other block's samples each
        const uint64_t other = pair_of(order_key(vb), (uint32_t)ib);
        uint32_t r = 0;
#pragma unroll
        for (int j = 0; j < kWave / 4; ++j) r += lane_u64(other, (w >> 2) * (kWave / 4) + j) < smine ? 1u : 0u;
        ranks[(w >> 1) * kSample + (w & 1) * kWave + lane] = (uint16_t)r;
    }
    lds_barrier();   // the keys stay in flight
    const uint32_t r0 = (uint32_t)(part * kSample / G), r1 = (uint32_t)((part + 1) * kSample / G);
    if (split && tid < kSample) {   // `smine` is sample tid here
        uint32_t r = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) r += ranks[j * kSample + tid];
        sorted_keys[r] = (uint32_t)(smine >> 32);
        if (r == r0) own64[0] = smine;
        if (r == r1) own64[1] = smine;
    }
    const bool staged = K1 > 0 && K1 < N;   // Stage I has a choice to make
    uint32_t lo = misc[kMBracket], hi = misc[kMBracket + 1];
    if (N > kWave) {
        const uint32_t wide = min(hi - lo, 0x40000000u) * 3u;
        if (rlo < 0) lo = lo > wide ? lo - wide : 0u;
        if (rhi > last) hi = hi < 0xffffffffu - wide ? hi + wide : 0xffffffffu;
    }
    const int sh = range_shift(lo, hi);

    // ---- keys to LDS, the first range's histogram -----------------------------------
    uint32_t nlo_s = 0, hi_s = 0, wave_below = 0;
    auto keep_keys = [&](auto single) {   // single: the range is one key, counted as in stage1_histogram
        constexpr bool ONE = decltype(single)::value;
        uint32_t one = 0;
#pragma unroll
        for (int u = 0; u < S; ++u) {
            const int i = u * kThreads + tid;
            if (i < N) {
                const uint32_t qi = order_key(vi[u]);
                ki[i] = qi;
                if constexpr (TWO) {
                    const uint32_t qs = order_key(vs[u]);
                    ks[i] = qs;
                    nlo_s = max(nlo_s, ~qs);
                    hi_s = max(hi_s, qs);
                }
                if (staged) {
                    wave_below += (uint32_t)__popcll(__ballot(qi < lo));   // lane 0 is in every tile's ballot
                    if constexpr (ONE) one += (uint32_t)__popcll(__ballot(qi == lo));
                    else if (qi - lo <= hi - lo) atomicAdd(&H[(qi - lo) >> sh], 1u);
                }
            }
        }
        if (ONE && lane == 0 && one) atomicAdd(&H[0], one);
    };
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(staged && lo == hi), 0))   // the same in every thread
        keep_keys(std::true_type{});
    else keep_keys(std::false_type{});
    if constexpr (TWO) {
        nlo_s = wave_max_u32(nlo_s);
        hi_s = wave_max_u32(hi_s);
        if (lane == 0) {
            slots[w] = nlo_s;
            slots[kW + w] = hi_s;
        }
    }
    Boundary bd{};
    if (staged) {
        uint32_t below, inside;
        stage1_scan(wave_below, (uint32_t)K1, H, misc, slots + 4 * kW, slots + 5 * kW, below, inside);
        bd = stage1_boundary(ki, N, (uint32_t)K1, lo, hi, below, inside, H, misc, slots + 4 * kW, slots + 5 * kW);
    } else {
        __syncthreads();
    }
    const uint32_t ksmin = TWO ? ~max_all(slots, lane) : 0u, ksmax = TWO ? max_all(slots + kW, lane) : 0u;

    // ---- a blank image: no order in Stage I, Stage II's keys equal, ranks are indices --
    // (512 images of 2880 tokens 23.1 us with the passes below, 15.4 without; other
    // images pay 0.1 us for the question)
    const size_t wbase = (size_t)(d.row_off >> 5) + 2 * (size_t)img;
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(ksmin == ksmax && (!staged || bd.need == 0u)), 0)) {
        if (part > 0) return;
        const Stride sp{(uint32_t)d.t, (uint32_t)R, (uint32_t)K2, a.stride_real != 0};
        uint32_t* imp_words = split ? a.gimp + wbase : bimp;
        uint32_t* sel_words = split ? a.gsel + wbase : bsel;
        for (int i0 = w * kWave; i0 < N; i0 += kThreads) {   // a tile of 64 tokens
            const int i = i0 + lane;
            const uint64_t imp = __ballot(i < K1 && i < N);
            const uint64_t pick = __ballot(i >= K1 && i < N && K2 > 0 && sp.picks((uint32_t)(i - K1)));
            const int word = (i0 >> 5) + lane;
            if (lane < 2 && word < (N + 31) / 32) {
                imp_words[word] = (uint32_t)(imp >> (32 * lane));
                sel_words[word] = (uint32_t)((imp | pick) >> (32 * lane));
            }
        }
        if (split) return;   // emit_kernel writes the output of a shared image
        __syncthreads();
        const int tw = tile_word(N);
        emit(a, d, tw >= 0 ? *reinterpret_cast<const uint64_t*>(bsel + tw) : 0ull,
             tw >= 0 ? *reinterpret_cast<const uint64_t*>(bimp + tw) : 0ull, slots + 6 * kW);
        return;
    }

    // ---- X^imp and the own tokens of X^rem ------------------------------------------
    // A share's end is a key, or a pair where the sampled key repeats (its
    // neighbours decide: the workgroups on both sides of it read the same).
    Share own_range{0ull, 0ull, !(split && part < G - 1)};
    bool exact = staged ? bd.tie || bd.hi == 0xffffffffu : K1 > 0;
    if (!staged) bd.hi = 0xffffffffu;   // hi + 1 = 0: no key is X^imp or a member
    auto share_end = [&](uint32_t r, uint64_t pair) {
        const uint32_t k = sorted_keys[r];
        const bool repeats = k == sorted_keys[r - 1] || k == sorted_keys[r + 1] || k == 0u;
        exact |= repeats;
        return repeats ? pair : pair_of(k, 0u);
    };
    if (split && part > 0) own_range.lo = share_end(r0, own64[0]);
    if (!own_range.open) own_range.hi = share_end(r1, own64[1]);
    uint32_t qlo = 0u, qhi = 0u;
    if constexpr (TWO) {   // value range of the buckets
        qlo = split ? sorted_keys[r0] : misc[kMQuant];
        qhi = split ? sorted_keys[min(r1, (uint32_t)kSample - 1u)] : misc[kMQuant + 1];
        // at the ends of X^rem, out to its own range unless outliers stretch that
        // (a share of few samples is narrow, and half of an outermost one lies beyond them)
        const float w0 = key_value(qhi) - key_value(qlo), far = (split ? (float)G : 1.5f) * w0;
        if (part == 0 && key_value(qlo) - key_value(ksmin) <= far) qlo = ksmin;
        if (own_range.open && key_value(ksmax) - key_value(qhi) <= far) qhi = ksmax;
    }
    const Bucketing bk = make_bucketing(qlo, qhi, ksmin, ksmax, kBuckets);
    uint64_t* members = reinterpret_cast<uint64_t*>(cur);
    const uint64_t imp_end = staged ? pair_of(bd.lo, bd.ilo) : K1 > 0 ? ~0ull : 0ull;
    uint32_t* imp_bits = !split || part == 0 ? bimp : nullptr;
    uint32_t own = 0, rem_below = 0;   // own: bit u, slot u
    auto pass = [&](auto ex) {
        second_pass<decltype(ex)::value, TWO>(ki, ks, N, bd, imp_end, staged, own_range, members, &misc[kMCount],
                                         imp_bits, split ? nullptr : bsel, own, rem_below);
    };
    if (__builtin_amdgcn_readfirstlane(exact)) pass(std::true_type{});   // the same in every thread
    else pass(std::false_type{});
    __syncthreads();
    int extra = -1;   // a boundary member that is an own token
    if (staged) {
        const uint32_t m = min(misc[kMCount], kMembers);
        if (tid < (int)m) {
            const uint64_t me = members[tid];
            const uint32_t i = (uint32_t)me;
            uint32_t r = 0;
            for (uint32_t j = 0; j < m; ++j) r += members[j] < me ? 1u : 0u;
            bool below = false;
            if (r < bd.need) {
                if (imp_bits) atomicOr(&bimp[i >> 5], 1u << (i & 31));
                if (!split) atomicOr(&bsel[i >> 5], 1u << (i & 31));
            } else if constexpr (TWO) {
                const uint64_t ps = pair_of(ks[i], i);
                below = ps < own_range.lo;
                if (!below && (own_range.open || ps < own_range.hi)) extra = (int)i;
            }
            if constexpr (TWO) rem_below += (uint32_t)__popcll(__ballot(below));   // lane 0 takes part if any lane does
        }
    }
    if (TWO && K2 > 0) {
        const Stride sp{(uint32_t)d.t, (uint32_t)R, (uint32_t)K2, a.stride_real != 0};
        uint32_t* pick = split ? a.gsel + wbase : bsel;
        auto keep = [&](uint32_t i) { atomicOr(&pick[i >> 5], 1u << (i & 31)); };
        auto for_own = [&](auto f) {   // every own token of this thread
            for (uint32_t o = own; o; o &= o - 1u) f((__ffs((int)o) - 1) * kThreads + tid);
            if (extra >= 0) f(extra);
        };
        if (__builtin_expect(bk.mode == 2, 0)) {   // one key, one bucket
            const uint32_t n = wave_sum_u32((uint32_t)__popc(own) + (extra >= 0 ? 1u : 0u));
            if (lane == 0 && n) atomicAdd(&H[0], n);
        } else {
            for_own([&](int i) { atomicAdd(&H[bucket_of(bk, ks[i], kBuckets)], 1u); });
        }
        __syncthreads();
        if (split && part == 0)
            for (int i = tid; i < (N + 31) / 32; i += kThreads) a.gimp[wbase + i] = bimp[i];
        const uint32_t c = H[tid];
        const uint32_t inc = wave_scan_add(c), sq = wave_sum_u32(c * c);   // at most N^2
        if (lane == kWave - 1) slots[w] = inc;
        if (lane == 0) {
            slots[kW + w] = sq;
            slots[2 * kW + w] = rem_below;
        }
        __syncthreads();
        const uint32_t start = inc - c + sum_before(slots, w, lane);
        const int m = (int)sum_before(slots, kW, lane);
        const uint32_t base = sum_before(slots + 2 * kW, kW, lane);
        const bool sorted = sum_before(slots + kW, kW, lane) > kCountFixed + kCountPer * (uint32_t)m;
        H[tid] = start;     // bucket starts and cursors from here on
        cur[tid] = start;
        __syncthreads();
        if (sorted) {
            // the tokens left out (G = 1: X^imp, as it is)
            const int words = 2 * ((N + kWave - 1) / kWave);
            if (split) {
                for (int i = tid; i < words; i += kThreads) bimp[i] = 0xffffffffu;
                __syncthreads();
                for_own([&](int i) { atomicAnd(&bimp[i >> 5], ~(1u << (i & 31))); });
            }
            __syncthreads();
            uint16_t* idx = reinterpret_cast<uint16_t*>(ki);
            const uint32_t top = ksmin ^ ksmax;   // bits above its highest are the same in every key
            const uint16_t* order = radix_sort(ks, bimp, N, m, top ? 0xffffffffu >> __clz((int)top) : 0u, idx, idx + N,
                                               reinterpret_cast<uint16_t*>(H), slots + 4 * kW, slots + 5 * kW);
            for (int j = tid; j < m; j += kThreads)
                if (sp.picks(base + (uint32_t)j)) keep(order[j]);
        } else {
            // The own tokens go to their buckets' cursors in the list, then a
            // thread per listed token counts the smaller members of its bucket.
            // PARTS: the buckets that start in [from, to), for the list holds
            // no more (an image above kListN that one workgroup ranks alone:
            // 17000 tokens in two parts 56 us, as one list of u16 indices 103).
            uint64_t* list = reinterpret_cast<uint64_t*>(smem + L.list);
            auto rank_part = [&](uint32_t from, uint32_t to, auto parts) {
                constexpr bool PARTS = decltype(parts)::value;
                for_own([&](int i) {
                    const int b = bucket_of(bk, ks[i], kBuckets);
                    if (PARTS && (H[b] < from || H[b] >= to)) return;
                    list[atomicAdd(&cur[b], 1u) - from] = pair_of(ks[i], (uint32_t)i);
                });
                __syncthreads();
                for (uint32_t j = from + (uint32_t)tid; j < to; j += kThreads) {
                    const uint64_t me = list[j - from];
                    const int b = bucket_of(bk, (uint32_t)(me >> 32), kBuckets);
                    const uint32_t beg = H[b];
                    if (sp.picks(base + from + rank_in(list, beg - from, cur[b] - beg, me))) keep((uint32_t)me);
                }
            };
            const uint32_t cap = (uint32_t)(L.list_bytes / 8), all = (uint32_t)m;
            if (all <= cap) {
                rank_part(0u, all, std::false_type{});
            } else {
                for (uint32_t from = 0, to; from < all; from = to) {
                    to = all;
                    if (all - from > cap) {   // the last bucket start within the list's reach
                        int b = 0;
                        for (int step = kBuckets / 2; step; step >>= 1)
                            if (H[b + step] <= from + cap) b += step;
                        to = H[b];
                        if (to <= from) break;   // a bucket that the list cannot hold: never (static_assert above)
                    }
                    rank_part(from, to, std::true_type{});
                    __syncthreads();
                }
            }
        }
    }
    if (split) return;   // emit_kernel writes the output of a shared image
    __syncthreads();
    const int tw = tile_word(N);
    emit(a, d, tw >= 0 ? *reinterpret_cast<const uint64_t*>(bsel + tw) : 0ull,
         tw >= 0 ? *reinterpret_cast<const uint64_t*>(bimp + tw) : 0ull, slots + 6 * kW);
}

// Output of the images select_kernel shared between workgroups: X^imp and the
// picks from the global bitmaps (which are cleared for the next call), then
// the ordered output (each lane reads its own tile's words).  One workgroup per
// image of the launch.
__global__ __launch_bounds__(kThreads) void emit_kernel(SelectArgs a)
{
    __shared__ uint32_t row[kW];
    const int G = a.groups > 0 ? a.groups : 1;
    const int local = (int)blockIdx.x;
    const int img = a.img0 + local;
    const Img d = image_of(a, local);
    const int N = d.n, K1 = d.k1, K2 = d.k2;
    if (!(G > 1 && K2 > 0 && N - K1 >= kShareRem)) return;   // emitted by select_kernel
    const size_t wbase = (size_t)(d.row_off >> 5) + 2 * (size_t)img;
    const int words = (N + 31) / 32, tw = tile_word(N);
    uint64_t sel = 0, imp = 0;
    if (tw >= 0) {
        const uint32_t* gi = a.gimp + wbase + tw;
        uint32_t* gs = a.gsel + wbase + tw;
        const bool two = tw + 1 < words;
        const uint32_t i0 = gi[0], s0 = gs[0], i1 = two ? gi[1] : 0u, s1 = two ? gs[1] : 0u;
        gs[0] = 0u;
        if (two) gs[1] = 0u;
        imp = (uint64_t)i1 << 32 | i0;
        sel = imp | ((uint64_t)s1 << 32 | s0);
    }
    emit(a, d, sel, imp, row);
}

// ---- images of at most kSmallSelectN tokens: one token per thread ------------
//
// Both stages are ranked in the same passes.  Every token gets its exact rank
// in (Stage II key, index) order among all N tokens, and its place relative
// to K1 in (Stage I key, index) order (counted exactly only inside the bucket
// that holds the K1 boundary); X^imp is the places below K1, and a token of X^rem
// ranks in X^rem as its Stage II rank minus the X^imp tokens ranked below it (read
// from a bitmap of X^imp in Stage II rank order), which decides the stride picks.
// Ranks come from value buckets and exact counting inside a bucket: bucket =
// clamp(floor((v - lo) nb / (hi - lo)), 0, nb - 1) is non-decreasing in the
// key, so rank = (tokens in lower buckets) + (members of the token's bucket
// smaller in (key, index) order).  lo and hi are about the 1.5 % and 98.5 %
// quantiles of a 64-key sample, so outliers (all-zero rows, zero-norm states)
// land in the two end buckets instead of crowding the bulk into a few; when
// the sample's range is not a finite positive float width, buckets are equal
// ranges of the order-preserving key itself.  All keys equal: rank = index.
// Phases are separated by eight workgroup barriers.  With a fused gather, G
// workgroups share an image: each repeats the selection and copies every G-th
// share of the kept rows (group 0 writes out_idx / out_src / out_rows).

struct SmallLayout {
    size_t hi, hs, si, ss, li, ls, samp, slots, misc, imps, kept, total;
};

__host__ __device__ inline SmallLayout small_layout(int T)
{
    SmallLayout L;
    size_t o = 0;
    L.hi = o;  o += 4 * (size_t)T;            // Stage I histogram, then cursors
    L.hs = o;  o += 4 * (size_t)T;            // Stage II histogram, then cursors
    L.si = o;  o += 4 * ((size_t)T + 1);      // Stage I bucket starts
    L.ss = o;  o += 4 * ((size_t)T + 1);      // Stage II bucket starts
    o = align_up(o, 16);
    L.li = o;  o += 8 * (size_t)T;            // (key << 32 | index) in Stage I bucket order
    L.ls = o;  o += 8 * (size_t)T;            // the same for Stage II
    L.samp = o; o += 8 * 128;                 // 64-key samples of both keys, (key << 6 | k)
    L.slots = o; o += 4 * 8 * kW;             // per-wavefront partial values
    L.misc = o; o += 4 * 16;                  // broadcast slots
    L.imps = o; o += 4 * 32;                  // X^imp bitmap in Stage II rank order
    L.kept = o; o += 4 * (size_t)T;           // token of each output slot (fused gather)
    L.total = o;
    return L;
}

typedef uint32_t u32x4s __attribute__((ext_vector_type(4)));
typedef u32x4s u32x4s_any __attribute__((aligned(2)));   // 16 bytes at any element

__global__ __launch_bounds__(kSmallSelectN) void select_small_kernel(SelectArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int T = (int)blockDim.x, nb = T, nw = T / kWave;
    const int G = a.ggroups > 0 ? a.ggroups : 1;
    const int local = (int)blockIdx.x / G, part = (int)blockIdx.x % G;
    const Img d = image_of(a, local);
    const int N = d.n, K1 = d.k1, K2 = d.k2, K = K1 + K2;
    const int tid = (int)threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const bool valid = tid < N;
    const SmallLayout L = small_layout(T);
    uint32_t* Hi = reinterpret_cast<uint32_t*>(smem + L.hi);
    uint32_t* Hs = reinterpret_cast<uint32_t*>(smem + L.hs);
    uint32_t* Si = reinterpret_cast<uint32_t*>(smem + L.si);
    uint32_t* Ss = reinterpret_cast<uint32_t*>(smem + L.ss);
    uint64_t* Li = reinterpret_cast<uint64_t*>(smem + L.li);
    uint64_t* Ls = reinterpret_cast<uint64_t*>(smem + L.ls);
    uint64_t* samp = reinterpret_cast<uint64_t*>(smem + L.samp);
    uint32_t* slots = reinterpret_cast<uint32_t*>(smem + L.slots);
    uint32_t* misc = reinterpret_cast<uint32_t*>(smem + L.misc);
    uint32_t* imps = reinterpret_cast<uint32_t*>(smem + L.imps);
    uint32_t* kept = reinterpret_cast<uint32_t*>(smem + L.kept);

    // ---- keys, samples, per-wavefront ranges ----------------------------------
    // every load in one burst: a token's keys, and in the wavefront that ranks it
    // a sample (every wavefront loading both: 30 images of 512 tokens 9.4 -> 9.9 us)
    const float* fi = a.key_imp + d.row_off;
    const float* fs = a.key_s + d.row_off;
    const int it = min(tid, N - 1), iq = sample_index(N, lane), iqc = min(iq, N - 1);
    const float vi = fi[it], vs = fs[it];
    float ui = 0.f, us = 0.f;
    const int wu = __builtin_amdgcn_readfirstlane(w), ws = nw > 1 ? 1 : 0;
    if (wu == 0) ui = fi[iqc];
    if (wu == ws) us = fs[iqc];
    const uint32_t ki = valid ? order_key(vi) : 0u, ks = valid ? order_key(vs) : 0u;
    // the quantiles of both keys, by wavefronts 0 and 1 (0 alone for N <= 64)
    const int q_lo = N > kWave ? 1 : 0, q_hi = N > kWave ? kWave - 2 : N - 1;
    if (wu == 0) sample_quantiles(iq < N ? order_key(ui) : 0xffffffffu, lane, samp, q_lo, q_hi, &misc[0]);
    if (wu == ws)
        sample_quantiles(iq < N ? order_key(us) : 0xffffffffu, lane, samp + kWave, q_lo, q_hi, &misc[2]);
    Hi[tid] = 0u;
    Hs[tid] = 0u;
    kept[tid] = 0xffffffffu;
    if (tid < 32) imps[tid] = 0u;
    {
        const uint32_t nlo_i = wave_max_u32(valid ? ~ki : 0u), hi_i = wave_max_u32(valid ? ki : 0u);
        const uint32_t nlo_s = wave_max_u32(valid ? ~ks : 0u), hi_s = wave_max_u32(valid ? ks : 0u);
        if (lane == 0) {
            slots[w] = nlo_i;
            slots[kW + w] = hi_i;
            slots[2 * kW + w] = nlo_s;
            slots[3 * kW + w] = hi_s;
        }
    }
    __syncthreads();   // B1
    auto max_of = [&](const uint32_t* row) { return wave_max_u32(lane < nw ? row[lane] : 0u); };
    const uint32_t kimin = ~max_of(slots), kimax = max_of(slots + kW);
    const uint32_t ksmin = ~max_of(slots + 2 * kW), ksmax = max_of(slots + 3 * kW);
    // Buckets over the sample quantiles (outliers clamp into the end buckets);
    // the histogram's atomic returns each token's place within its bucket.
    const Bucketing bi = make_bucketing(misc[0], misc[1], kimin, kimax, nb);
    const Bucketing bs = make_bucketing(misc[2], misc[3], ksmin, ksmax, nb);
    const int gi = valid ? bucket_of(bi, ki, nb) : 0;
    const int gs = valid ? bucket_of(bs, ks, nb) : 0;
    uint32_t li = 0, ls = 0;
    if (valid) {
        li = atomicAdd(&Hi[gi], 1u);
        ls = atomicAdd(&Hs[gs], 1u);
    }
    __syncthreads();   // B2
    // ---- bucket starts: thread t owns bucket t ----------------------------------
    const uint32_t ci = Hi[tid], cs = Hs[tid];
    const uint32_t inc_i = wave_scan_add(ci), inc_s = wave_scan_add(cs);
    if (lane == kWave - 1) {
        slots[4 * kW + w] = inc_i;
        slots[5 * kW + w] = inc_s;
    }
    __syncthreads();   // B3
    Si[tid] = inc_i - ci + sum_before(slots + 4 * kW, w, lane);
    Ss[tid] = inc_s - cs + sum_before(slots + 5 * kW, w, lane);
    if (tid == T - 1) {
        Si[T] = (uint32_t)N;
        Ss[T] = (uint32_t)N;
    }
    __syncthreads();   // B4
    // ---- members of shared buckets listed; exact ranks ------------------------
    const uint64_t me_i = ((uint64_t)ki << 32) | (uint32_t)tid;
    const uint64_t me_s = ((uint64_t)ks << 32) | (uint32_t)tid;
    uint32_t bi0 = 0, bi1 = 0, bs0 = 0, bs1 = 0;
    if (valid) {
        bi0 = Si[gi];
        bi1 = Si[gi + 1];
        bs0 = Ss[gs];
        bs1 = Ss[gs + 1];
        // Stage I needs exact ranks only in the bucket that holds the K1
        // boundary: a lower bucket's members are all in X^imp, a higher
        // one's all out, whatever their order inside it.
        if (bi1 - bi0 > 1u && bi0 < (uint32_t)K1 && bi1 > (uint32_t)K1) Li[bi0 + li] = me_i;
        if (bs1 - bs0 > 1u) Ls[bs0 + ls] = me_s;
    }
    __syncthreads();   // B5
    uint32_t ri = bi0, rs = bs0;
    if (valid) {
        if (bi.mode == 2) ri = (uint32_t)tid;
        else if (bi1 - bi0 > 1u && bi0 < (uint32_t)K1 && bi1 > (uint32_t)K1) ri = rank_in(Li, bi0, bi1 - bi0, me_i);
        if (bs.mode == 2) rs = (uint32_t)tid;
        else if (bs1 - bs0 > 1u) rs = rank_in(Ls, bs0, bs1 - bs0, me_s);
        rs = rs < (uint32_t)N ? rs : (uint32_t)N - 1u;   // a rank below N in every case (memory safety)
    }
    const bool imp = valid && ri < (uint32_t)K1;
    if (imp && K2 > 0) atomicOr(&imps[rs >> 5], 1u << (rs & 31));
    __syncthreads();   // B6
    // ---- stride picks on the rank in X^rem, union, output slots -------------------
    // X^imp tokens ranked below rs: a wave scan of the bitmap words' counts
    // (lane q holds word q), then the partial word.
    const uint32_t wc = lane < 32 ? (uint32_t)__popc(imps[lane]) : 0u;
    const uint32_t wex = wave_scan_add(wc) - wc;
    const uint32_t wbelow = (uint32_t)__shfl((int)wex, (int)(rs >> 5));   // every lane takes part
    bool pick = false;
    if (valid && !imp && K2 > 0) {
        const uint32_t below = wbelow + (uint32_t)__popc(imps[rs >> 5] & ((1u << (rs & 31)) - 1u));
        const Stride sp{(uint32_t)d.t, (uint32_t)(N - K1), (uint32_t)K2, a.stride_real != 0};
        pick = sp.picks(rs - below);
    }
    const bool sel = imp || pick;
    const uint64_t bm = __ballot(sel);
    if (lane == 0) slots[6 * kW + w] = (uint32_t)__popcll(bm);
    __syncthreads();   // B7
    const uint32_t slot = sum_before(slots + 6 * kW, w, lane) + (uint32_t)__popcll(bm & lanes_below(lane));
    if (sel && slot < (uint32_t)K) {   // never more than K writes, whatever the keys
        if (part == 0) {
            const int o = d.out_off + (int)slot;
            a.out_idx[o] = tid;
            if (a.out_src) a.out_src[o] = imp ? 0 : 1;
            if (a.out_rows) a.out_rows[o] = d.row_off + tid;
        }
        kept[slot] = (uint32_t)tid;
    }
    if (!a.gX) return;
    __syncthreads();   // B8
    // ---- fused gather: this group's share of the kept rows -------------------------
    const int s0 = (int)(((int64_t)part * K) / G), s1 = (int)(((int64_t)(part + 1) * K) / G);
    const char* X = static_cast<const char*>(a.gX);
    char* out = static_cast<char*>(a.gout);
    const int64_t rb = a.grow_bytes;
    if (rb >= 16) {
        // Pieces of 16 bytes; a row's last one is its last 16 bytes (they
        // overlap the piece before when the row is no multiple of 16).  Piece j =
        // r * cpr + c of the share, walked with (r, c) carried
        // from step to step (no division per chunk).
        const uint32_t cpr = (uint32_t)((rb + 15) / 16), last = (uint32_t)(rb - 16);
        const uint32_t rows = (uint32_t)(s1 - s0);
        const uint32_t qT = (uint32_t)T / cpr, mT = (uint32_t)T % cpr;
        uint32_t r = (uint32_t)tid / cpr, c = (uint32_t)tid % cpr;
        constexpr int kUnr = 8;
        while (r < rows) {
            u32x4s v[kUnr];
            uint32_t rr[kUnr], cc[kUnr];
#pragma unroll
            for (int u = 0; u < kUnr; ++u) {
                rr[u] = r;
                cc[u] = c;
                if (r < rows) {
                    const uint32_t k = kept[s0 + (int)r];
                    const uint32_t tk = k < (uint32_t)N ? k : 0u;   // always a filled slot
                    v[u] = __builtin_nontemporal_load(
                        reinterpret_cast<const u32x4s_any*>(X + (int64_t)(d.row_off + (int)tk) * rb + min(c * 16, last)));
                }
                c += mT;
                r += qT;
                if (c >= cpr) {
                    c -= cpr;
                    ++r;
                }
            }
#pragma unroll
            for (int u = 0; u < kUnr; ++u) {
                if (rr[u] < rows)
                    __builtin_nontemporal_store(
                        v[u], reinterpret_cast<u32x4s_any*>(out + (int64_t)(d.out_off + s0 + (int)rr[u]) * rb +
                                                            min(cc[u] * 16, last)));
            }
        }
    } else if (a.gelem == 2) {
        const int64_t epr = rb / 2;
        for (int r = s0; r < s1; ++r) {
            const uint32_t tk = kept[r] < (uint32_t)N ? kept[r] : 0u;
            const uint16_t* src = reinterpret_cast<const uint16_t*>(X + (int64_t)(d.row_off + (int)tk) * rb);
            uint16_t* dst = reinterpret_cast<uint16_t*>(out + (int64_t)(d.out_off + r) * rb);
            for (int64_t c = tid; c < epr; c += T) dst[c] = src[c];
        }
    } else {
        const int64_t epr = rb / 4;
        for (int r = s0; r < s1; ++r) {
            const uint32_t tk = kept[r] < (uint32_t)N ? kept[r] : 0u;
            const uint32_t* src = reinterpret_cast<const uint32_t*>(X + (int64_t)(d.row_off + (int)tk) * rb);
            uint32_t* dst = reinterpret_cast<uint32_t*>(out + (int64_t)(d.out_off + r) * rb);
            for (int64_t c = tid; c < epr; c += T) dst[c] = src[c];
        }
    }
}

}  // namespace

int select_threads(int nmax)
{
    (void)nmax;
    return kThreads;
}

bool select_shares(const ImageDesc& d)
{
    return d.k2 > 0 && d.n - d.k1 >= kShareRem;
}

int select_groups(int64_t n_large, int cus)
{
    if (n_large <= 0) return 1;
    int g = 1;
    while (g < kMaxSplitGroups && n_large * 2 * g <= (int64_t)cus) g *= 2;
    return g;
}

size_t select_gsel_words(int64_t max_tokens, int max_images)
{
    return (size_t)(max_tokens / 32) + 2 * (size_t)max_images + 2;
}

size_t select_lds_bytes(int n, int threads)
{
    (void)threads;
    return n <= kMaxSlots * kThreads ? launch_lds(n) : SIZE_MAX;
}

hipError_t select_prepare(int lds_limit)
{
    for (auto kernel : {select_kernel<4, true>, select_kernel<10, true>, select_kernel<kMaxSlots, true>,
                        select_kernel<4, false>, select_kernel<10, false>, select_kernel<kMaxSlots, false>}) {
        const void* k = reinterpret_cast<const void*>(kernel);
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, lds_limit);
        if (e != hipSuccess) return e;
    }
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&select_small_kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, lds_limit);
}

int select_small_groups(int images, int k_min, int cus)
{
    // enough workgroups to keep every compute unit copying, at most one per
    // kept row and 16 per image
    int g = (2 * cus + images - 1) / (images > 0 ? images : 1);
    if (g > 16) g = 16;
    if (g > k_min) g = k_min;
    return g < 1 ? 1 : g;
}

hipError_t launch_select(const SelectArgs& a, int nmax, hipStream_t s)
{
    if (a.nimg <= 0) return hipSuccess;
    if (nmax <= kSmallSelectN) {
        const int T = ((nmax > kWave ? nmax : kWave) + kWave - 1) / kWave * kWave;
        const int G = a.gX && a.ggroups > 0 ? a.ggroups : 1;
        SelectArgs b = a;
        b.ggroups = G;
        hipLaunchKernelGGL(select_small_kernel, dim3(a.nimg * G), dim3(T), small_layout(T).total, s, b);
        return hipGetLastError();
    }
    bool two = false;
    for (int b = 0; b < (a.uniform ? 1 : a.nimg); ++b) two = two || a.desc[b].k2 > 0;
    const size_t lds = launch_lds(nmax, two);
    const int groups = two && a.groups > 0 ? a.groups : 1;
    auto pick = [&](auto stage2) {
        constexpr bool TWO = decltype(stage2)::value;
        return nmax <= 4 * kThreads ? select_kernel<4, TWO>
               : nmax <= 10 * kThreads ? select_kernel<10, TWO> : select_kernel<kMaxSlots, TWO>;
    };
    auto kernel = two ? pick(std::true_type{}) : pick(std::false_type{});
    hipLaunchKernelGGL(kernel, dim3(a.nimg * groups), dim3(kThreads), lds, s, a);
    if (groups > 1) {
        hipLaunchKernelGGL(emit_kernel, dim3(a.nimg), dim3(kThreads), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace tr
