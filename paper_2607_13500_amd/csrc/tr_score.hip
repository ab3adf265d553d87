// Fused per-token scoring: one HBM pass over X, X_pre and X_post.
//
// One wavefront scores one token row.  The row is cut into chunks of 16 bytes
// (8 bf16 or 4 fp32 elements); chunk c belongs to lane c % 64 and every lane
// walks its chunks in ascending c, so a row's arithmetic never depends on
// where the row sits in the batch (identical rows score identically).
//
// Eq. (3)-(4): with m = mean |x| and V = M2 / D (M2 = sum (|x| - m)^2),
//   sum_j p_j^2 = (1 + V / m^2) / D,  H2 = log D - log1p(CV^2),
//   CV^2 = M2 / (D m^2).
// Stage I ranks ascending CV^2 (= descending H2): near-uniform rows have H2
// within an fp32 ulp of log D but well-separated CV^2.  M2 is accumulated
// around one shift c shared by the whole row, the mean |x| of its first
// min(D, 64 * 16 / elem) elements (every lane's first chunk, summed by a
// butterfly before any other work): d = |x| - c is exact when |x| is within a
// factor 2 of c (near-uniform rows), and M2 = sum d^2 - (sum d)^2 / D has
// little cancellation because c lies close to m.
//
// Range: both scores are invariant to scaling a row by a positive constant
// (Eq. 3 divides by sum |x|, Eq. 6 by both norms), so X is scored as
// |x| 2^-e with 2^e the binade of the probe mean: the power of two is applied
// by the same fused multiply-add that subtracts the shift (exact for normal
// values, no extra instruction), and the sums of squares stay far from fp32
// overflow and underflow whatever the row's magnitude.  A row whose probe
// mean lies outside [2^-120, 2^120] (an all-zero probe included) or whose
// scaled sums leave [0, 2^100] is scored again from a second read of its
// bytes, scaled from its exact maximum |x| and shifted by its exact mean.
//
// Eq. (6): fp32 sums of x'x'', x'^2 and x''^2 (bf16 rows: hardware bf16 dot
// products of element pairs, accumulated in fp32), unscaled.  When both
// squared norms lie in [2^-60, FLT_MAX], products that underflow (or
// denormal inputs) move s by less than 2^-40 and nothing overflowed; any
// other row is scored again from a second read, each of x' and x'' scaled by
// the power of two of its own maximum |x|, in fp32 fused multiply-adds.
//
// Non-finite elements: a NaN or an infinity makes the first pass's sums NaN
// or infinite, so such a row always takes the second read, which is where it
// is detected; with a count requested, lane 0 adds one per such row.
//
// Lane partial sums are combined by a fixed DPP scan tree (the total is read
// from lane 63 into every lane) and lane 0 writes the results.
//
// A launch may compute only one of the two scores (Stage I's key alone, or
// Stage II's alone): the other tensor is then never read and its key is
// written as 0.  The scores that are computed are bit-identical to those of a
// launch that computes both, because each score's arithmetic is independent.
//
// Shannon variant of Stage I (H1 = -sum p log p of the same p): the key is
// KL = log D - H1 >= 0 (ascending = descending H1), accumulated without
// cancellation as a sum of non-negative terms.  With u = |x| / c for the same
// row shift c and g(u) = u log u - u + 1 >= 0, and r = mean|x| / c,
//   D KL = sum_j (|x_j|/m) log(|x_j|/m) = (sum_j g(u_j) - D g(r)) / r,
// where the subtracted D g(r) is small because c lies close to the mean.
// Every u is formed as 1 + e with e = (|x| - c) (1/c) + delta, delta =
// c (1/c) - 1 taken exactly by a fused multiply-add, so all terms (and r)
// refer to the same effective shift 1 / (1/c) and e keeps full relative
// accuracy for near-uniform rows.  The terms are summed in base-2 units
// (e / ln 2 and g / ln 2), which saves a multiply per element; the row's sum
// is scaled by ln 2 once.
#include <type_traits>

#include "tr_row.h"
#include "tr_score.h"
#include "tr_wave.h"

namespace tr {
namespace {

// 16 bytes of raw row data.
struct Raw {
    uint32_t w[4];
};

template <bool BF16>
struct Layout {
    static constexpr int kV = BF16 ? 8 : 4;    // elements per 16-byte chunk
    static constexpr int kEB = BF16 ? 2 : 4;   // bytes per element
};

// bf16 -> fp32 is exact: the stored half is the upper half of the binary32.
__device__ __forceinline__ float lo_bf16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_bf16(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

template <bool BF16>
__device__ __forceinline__ void unpack(const Raw& r, float* v)
{
    if constexpr (BF16) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[2 * k] = lo_bf16(r.w[k]);
            v[2 * k + 1] = hi_bf16(r.w[k]);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = __uint_as_float(r.w[k]);
    }
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(2)));   // 16 bytes at any element

// The 16 bytes at byte `off` of a row.  Every byte is read exactly once, so the
// loads are non-temporal (streamed past the caches: measured 7.0 vs 6.2 TB/s
// for this access pattern on MI355X).  A row may start at any element: the
// 16-byte global load takes any byte address.
__device__ __forceinline__ Raw load16(const char* row, uint32_t off)
{
    Raw r;
    const u32x4 q = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(row + off));
    r.w[0] = q.x;
    r.w[1] = q.y;
    r.w[2] = q.z;
    r.w[3] = q.w;
    return r;
}

// A whole row of m elements, fewer than a chunk holds, zero-padded.
template <bool BF16>
__device__ __forceinline__ Raw load_short(const char* row, int m)
{
    Raw r{{0u, 0u, 0u, 0u}};
    if constexpr (BF16) {
        const uint16_t* e = reinterpret_cast<const uint16_t*>(row);
#pragma unroll
        for (int k = 0; k < 7; ++k)
            if (k < m) r.w[k >> 1] |= (uint32_t)e[k] << (16 * (k & 1));
    } else {
        const uint32_t* e = reinterpret_cast<const uint32_t*>(row);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (k < m) r.w[k] = e[k];
    }
    return r;
}

// The last m elements of a row's last 16 bytes, moved to the front and
// zero-padded: the row's partial chunk (m is the same for every row).
template <bool BF16>
__device__ __forceinline__ Raw tail_of(Raw r, int m)
{
    int words = Layout<BF16>::kV - m;   // leading elements, which belong to the chunk before
    if constexpr (BF16) {
        if (words & 1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) r.w[k] = (r.w[k] >> 16) | (k < 3 ? r.w[k + 1] << 16 : 0u);
        }
        words >>= 1;
    }
    if (words & 1) {
#pragma unroll
        for (int k = 0; k < 4; ++k) r.w[k] = k < 3 ? r.w[k + 1] : 0u;
    }
    if (words & 2) {
        r.w[0] = r.w[2];
        r.w[1] = r.w[3];
        r.w[2] = r.w[3] = 0u;
    }
    return r;
}

struct XAcc {
    float sd;    // sum (|x| 2^-e - c)
    float sd2;   // sum (|x| 2^-e - c)^2; Shannon: sum g(|x| 2^-e / c) / ln 2
};

struct CAcc {
    float dot, n1, n2;
};

// d = |x| 2^-e - c in one fused multiply-add (scale = 2^-e): the product is
// exact for normal values, so d is the rounding of the exact scaled
// difference, and for near-uniform rows exact (Sterbenz).
template <int V>
__device__ __forceinline__ void x_chunk(XAcc& a, const float* v, int m, float c, float scale)
{
#pragma unroll
    for (int k = 0; k < V; ++k) {
        if (k >= m) continue;
        const float d = fmaf(fabsf(v[k]), scale, -c);
        a.sd += d;
        a.sd2 = fmaf(d, d, a.sd2);
    }
}

// Base-2 units: y = e / ln 2 and g2(y) = g(1 + e) / ln 2 >= 0, given y (and
// u = 1 + e for the direct form); the row's sum is multiplied by ln 2 once.
// For |e| < 1/4 as y^2 psi(y), psi a degree-5 polynomial (the Chebyshev
// interpolant of g(1 + e) / (y^2 ln 2) on |y| < (1/4) / ln 2, relative error
// 3e-7, 4e-7 with fp32 Horner; coefficients from gen_shannon_poly.py), which
// keeps full relative accuracy where the direct form cancels (in fp32 the
// direct form's error grows to 1e-5 at |e| = 1/8, so the cut stays at 1/4);
// elsewhere u log2 u - y with the hardware base-2 logarithm (argument clamped
// to 1e-30, a normal number, so u = 0 gives 0 - y = 1 / ln 2).  Both forms
// are evaluated and one is selected: no per-element divergence.
constexpr float kInvLn2 = 1.44269504088896340736f;
constexpr float kLn2 = 0.693147180559945309f;
constexpr float kShannonCut = 0.25f * kInvLn2;   // |e| < 1/4 in units of y

__device__ __forceinline__ float g2_shannon(float y, float u)
{
    float p = -2.818413918e-03f;
    p = fmaf(p, y, 5.614020020e-03f);
    p = fmaf(p, y, -1.152998215e-02f);
    p = fmaf(p, y, 2.773815429e-02f);
    p = fmaf(p, y, -8.007569547e-02f);
    p = fmaf(p, y, 3.465736915e-01f);
    const float series = (y * y) * p;
    const float direct = fmaf(u, __builtin_amdgcn_logf(fmaxf(u, 1e-30f)), -y);
    return fabsf(y) < kShannonCut ? series : direct;
}

// Shannon partial sums over m elements for a row shift c > 0 and scale
// 2^-e (inv_u = 2^-e / c, u = |x| inv_u; inv2 = (1/c) / ln 2 and delta2 =
// (c (1/c) - 1) / ln 2 give y): sd as for CV^2, sd2 = sum g(u) / ln 2.
template <int V>
__device__ __forceinline__ void x_chunk_shannon(XAcc& a, const float* v, int m, float c, float scale,
                                                float inv_u, float inv2, float delta2)
{
#pragma unroll
    for (int k = 0; k < V; ++k) {
        if (k >= m) continue;
        const float ax = fabsf(v[k]);
        const float d = fmaf(ax, scale, -c);
        a.sd += d;
        a.sd2 += g2_shannon(fmaf(d, inv2, delta2), ax * inv_u);
    }
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b),
                                           c, false);
}

// Eq. (6) partial sums over one chunk.  bf16: the hardware dot product of the
// two bf16 pairs in each 32-bit word (products of bf16 values are exact in
// fp32), no unpacking; fp32: fused multiply-adds.  Unused elements of a
// partial chunk are zero and add nothing.
template <bool BF16>
__device__ __forceinline__ void c_chunk(CAcc& a, const Raw& p, const Raw& q)
{
    if constexpr (BF16) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            a.dot = dot2_bf16(p.w[k], q.w[k], a.dot);
            a.n1 = dot2_bf16(p.w[k], p.w[k], a.n1);
            a.n2 = dot2_bf16(q.w[k], q.w[k], a.n2);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float u = __uint_as_float(p.w[k]), v = __uint_as_float(q.w[k]);
            a.dot = fmaf(u, v, a.dot);
            a.n1 = fmaf(u, u, a.n1);
            a.n2 = fmaf(v, v, a.n2);
        }
    }
}

__device__ __forceinline__ float wave_sum(float v) { return wave_sum_f32(v); }

// The row shift c of the scaled values and what the Shannon terms derive
// from it (1/c and its rounding offset, folded with the scale).
struct Shift {
    float c, scale, inv_c, delta, inv_u, inv2, delta2;
};

__device__ __forceinline__ Shift make_shift(float c, float scale)
{
    Shift h;
    h.c = c;
    h.scale = scale;
    h.inv_c = c > 0.f ? 1.f / c : 0.f;
    h.delta = c > 0.f ? fmaf(c, h.inv_c, -1.f) : 0.f;
    h.inv_u = h.inv_c * scale;
    h.inv2 = h.inv_c * kInvLn2;
    h.delta2 = h.delta * kInvLn2;
    return h;
}

template <bool H1, int V>
__device__ __forceinline__ void x_accumulate(XAcc& xa, const float* v, int m, const Shift& h)
{
    if constexpr (H1) x_chunk_shannon<V>(xa, v, m, h.c, h.scale, h.inv_u, h.inv2, h.delta2);
    else x_chunk<V>(xa, v, m, h.c, h.scale);
}

// Stage I sums of a row from a second read of its bytes: scaled by the power
// of two of its exact maximum |x| and shifted by its exact scaled mean, so
// that no term can overflow and none that matters underflows.  zero: every
// element is 0 (or the row is not finite).
struct XRow {
    Shift h;
    float sd, sd2;
    bool zero;
    bool nonfinite;   // some element is a NaN or infinite
};

template <bool BF16, bool H1>
__device__ __noinline__ XRow x_reread(const char* row, int D, int lane)
{
    XRow r;
    r.sd = r.sd2 = 0.f;
    float mx = 0.f, mn = __builtin_inff();
    bool bad = false;
    for (int j = lane; j < D; j += kWave) {
        const float a = fabsf(elem<BF16>(row, j));
        mx = fmaxf(mx, a);
        mn = fminf(mn, a);
        bad = bad || !(a <= 3.40282347e38f);   // NaN or infinite
    }
    const float rmax = wave_max_nonneg(mx);
    const float rmin = wave_min_nonneg(mn);
    r.nonfinite = __any(bad) != 0;
    r.zero = !(rmax > 0.f && rmax <= 3.40282347e38f);
    if (r.zero) {
        r.h = make_shift(0.f, 1.f);
        return r;
    }
    // The values are scaled once here (exact: the results are normal or
    // negligibly small), so the Shannon terms' 1/c is never folded with the
    // scale, which for a tiny row could leave the fp32 range.
    const float scale = binade_scale(rmax);
    float sum = 0.f;
    for (int j = lane; j < D; j += kWave) sum += fabsf(elem<BF16>(row, j)) * scale;
    // (a row of one magnitude: that magnitude, exactly, as the shift)
    r.h = make_shift(rmin == rmax ? rmax * scale : wave_sum(sum) / (float)D, 1.f);
    XAcc xa{0.f, 0.f};
    for (int j = lane; j < D; j += kWave) {
        const float v = elem<BF16>(row, j) * scale;
        x_accumulate<H1, 1>(xa, &v, 1, r.h);
    }
    r.sd = wave_sum(xa.sd);
    r.sd2 = wave_sum(xa.sd2);
    return r;
}

// How a launch reads its rows.
constexpr int kBurst = 0;   // up to four chunks of every tensor per lane at once
constexpr int kPaced = 1;   // one or two loads of a wavefront in flight (see launch_t)
constexpr int kOdd = 2;     // as kBurst; rows that are no whole number of 16-byte chunks

template <int N>
using Int = std::integral_constant<int, N>;

template <bool BF16, int MODE, int READ>
__global__ __launch_bounds__(kWave) void score_kernel(ScoreArgs a)
{
    using L = Layout<BF16>;
    constexpr int V = L::kV;
    constexpr bool kX = (MODE & kScoreImp) != 0;    // Eq. (3)-(4) over X
    constexpr bool kC = (MODE & kScoreSim) != 0;    // Eq. (6) over X_pre, X_post
    constexpr bool kH1 = kX && (MODE & kScoreShannon) != 0;   // Shannon variant of Stage I
    constexpr bool ODD = READ == kOdd;
    // Paced reads: wait for the loads before, so X_pre and X_post go out
    // together after X's chunk, or singly when they are all that is read.
    [[maybe_unused]] auto pace = [] {
        if constexpr (READ == kPaced) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    const int lane = threadIdx.x;
    const int64_t row = blockIdx.x;

    const char* xr = static_cast<const char*>(a.X) + row * (int64_t)a.D * L::kEB;
    const char* pr = static_cast<const char*>(a.P) + row * (int64_t)a.Dc * L::kEB;
    const char* qr = static_cast<const char*>(a.Q) + row * (int64_t)a.Dc * L::kEB;
    // Whole chunks, and the elements of a trailing partial chunk.  That one
    // belongs to lane (index % 64) like any other and is its lane's last.
    const int nfx = kX ? a.D / V : 0, mx = kX && ODD ? a.D % V : 0;
    const int nfc = kC ? a.Dc / V : 0, mc = kC && ODD ? a.Dc % V : 0;
    // A column is 64 chunks, one to a lane.
    const int colsx = (nfx + (mx ? 1 : 0) + kWave - 1) / kWave, colsc = (nfc + (mc ? 1 : 0) + kWave - 1) / kWave;
    const int endx = a.D * L::kEB - 16, endc = a.Dc * L::kEB - 16;   // a row's last 16 bytes
    const bool short_rows = ODD && ((kX && endx < 0) || (kC && endc < 0));
    // elements in the lanes' first chunks: the sample the shift c averages
    const float n_probe = (float)(a.D < kWave * V ? a.D : kWave * V);

    XAcc xa{0.f, 0.f};
    CAcc ca{0.f, 0.f, 0.f};
    // The shift and scale from the probe mean (wave-uniform): the row is
    // accumulated as |x| 2^-e with the probe mean in [0.5, 1) after scaling.
    Shift sh = make_shift(0.f, 1.f);
    bool fast_x = false;
    // The probe is this lane's first m elements pv (lane 0 always has some).
    // Its mean is the shift; when every probe element has one magnitude, that
    // magnitude itself is (exact, so an exactly uniform row gets d = 0 and a
    // key of exactly 0 whatever its magnitude).  Either way c is a mean or a
    // value of a subset of the row, which bounds the cancellation in M2.
    auto set_probe = [&](const float* pv, int m) {
        const float ref = __uint_as_float(
            (uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(fabsf(pv[0])), 0));
        bool same = true;
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < V; ++k) {
            if (k >= m) continue;
            sum += fabsf(pv[k]);
            same = same && fabsf(pv[k]) == ref;
        }
        const float c_raw = __all(same) ? ref : wave_sum(sum) / n_probe;
        fast_x = c_raw >= 0x1p-120f && c_raw <= 0x1p120f;
        const float scale = fast_x ? binade_scale(c_raw) : 1.f;
        sh = make_shift(fast_x ? c_raw * scale : 0.f, scale);
    };
    // One step: UNR columns from column c0 on, of X (HX) and of X_pre and X_post
    // (HC).  Every load of a step is issued before anything waits: a lane past
    // the row's end loads its last 16 bytes (the wavefront's lanes then ask for
    // one address) instead of skipping the load.  Skipped loads kept their
    // registers tied to the step before, so the loads went out one or two at a
    // time, each behind the one before.  The lane of a partial chunk gets it
    // at the end of those 16 bytes.
    auto step = [&](int c0, auto unr, auto has_x, auto has_c) __attribute__((always_inline)) {
        constexpr int UNR = decltype(unr)::value;
        constexpr bool HX = decltype(has_x)::value, HC = decltype(has_c)::value;
        const int j0 = c0 * kWave;
        [[maybe_unused]] Raw rx[UNR], rp[UNR], rq[UNR];
        if (!short_rows) {
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const uint32_t off = (uint32_t)(j0 + lane + kWave * u) * 16;
                if constexpr (HX) {
                    pace();
                    rx[u] = load16(xr, min(off, (uint32_t)endx));
                }
                if constexpr (HC) {
                    pace();
                    rp[u] = load16(pr, min(off, (uint32_t)endc));
                    if constexpr (!HX) pace();
                    rq[u] = load16(qr, min(off, (uint32_t)endc));
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const uint32_t off = (uint32_t)(j0 + lane + kWave * u) * 16;
                if constexpr (HX) rx[u] = endx < 0 ? load_short<BF16>(xr, mx) : load16(xr, min(off, (uint32_t)endx));
                if constexpr (HC) {
                    rp[u] = endc < 0 ? load_short<BF16>(pr, mc) : load16(pr, min(off, (uint32_t)endc));
                    rq[u] = endc < 0 ? load_short<BF16>(qr, mc) : load16(qr, min(off, (uint32_t)endc));
                }
            }
        }
        asm volatile("" ::: "memory");   // the loads stay here, none moves down to its use
        if (HX && c0 == 0) {
            float v[V];
            int m = 0;
            v[0] = 0.f;
            if (lane < nfx) {
                unpack<BF16>(rx[0], v);
                m = V;
            } else if (ODD && lane == nfx && mx) {
                unpack<BF16>(endx < 0 ? rx[0] : tail_of<BF16>(rx[0], mx), v);
                m = mx;
            }
            set_probe(v, m);
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int ci = j0 + lane + kWave * u;
            if (HX && ci < nfx) {
                float v[V];
                unpack<BF16>(rx[u], v);
                x_accumulate<kH1, V>(xa, v, V, sh);
            }
            if (HC && ci < nfc) c_chunk<BF16>(ca, rp[u], rq[u]);
            if constexpr (ODD) {
                if (HX && mx && ci == nfx) {
                    float v[V];
                    unpack<BF16>(endx < 0 ? rx[u] : tail_of<BF16>(rx[u], mx), v);
                    x_accumulate<kH1, V>(xa, v, mx, sh);
                }
                if (HC && mc && ci == nfc)
                    c_chunk<BF16>(ca, endc < 0 ? rp[u] : tail_of<BF16>(rp[u], mc),
                                  endc < 0 ? rq[u] : tail_of<BF16>(rq[u], mc));
            }
        }
    };
    // Columns from .. to - 1 in steps of four (paced: one) and a last one of
    // exactly what is left: loads past the row, all of one address, still cost
    // as much as others (300000 rows of 257 bf16 elements in steps of four 436 us).
    auto run = [&](int from, int to, auto has_x, auto has_c) __attribute__((always_inline)) {
        int c = from;
        if constexpr (READ == kPaced) {
            for (; c < to; ++c) step(c, Int<1>{}, has_x, has_c);
        } else {
            for (; to - c >= 4; c += 4) step(c, Int<4>{}, has_x, has_c);
            const int rest = to - c;
            if (rest == 2) step(c, Int<2>{}, has_x, has_c);
            else if (rest == 1) step(c, Int<1>{}, has_x, has_c);
            else if (rest == 3) step(c, Int<3>{}, has_x, has_c);
        }
    };
    if constexpr (kX && kC) {
        const int both = min(colsx, colsc);
        run(0, both, std::true_type{}, std::true_type{});
        if (colsx != colsc) {
            if (colsx > both) run(both, colsx, std::true_type{}, std::false_type{});
            else run(both, colsc, std::false_type{}, std::true_type{});
        }
    } else {
        run(0, kX ? colsx : colsc, std::bool_constant<kX>{}, std::bool_constant<kC>{});
    }

    float sd = 0.f, sd2 = 0.f, s = 0.f;
    bool zero_row = false;
    // A NaN or infinite element always sends its row to a second read (its
    // sums leave the range the first pass accepts), which reports it.
    bool bad_row = false;
    if constexpr (kX) {
        sd = wave_sum(xa.sd);
        sd2 = wave_sum(xa.sd2);
        // Probe outside the window, or a scaled sum out of range (NaN too):
        // score the row again from its maximum (a wave-uniform decision).
        if (!(fast_x && sd2 <= 0x1p100f)) {
            const XRow r = x_reread<BF16, kH1>(xr, a.D, lane);
            bad_row = r.nonfinite;
            sh = r.h;
            sd = r.sd;
            sd2 = r.sd2;
            zero_row = r.zero;
        }
    }
    if constexpr (kC) {
        const float dot = wave_sum(ca.dot), n1 = wave_sum(ca.n1), n2 = wave_sum(ca.n2);
        if (cos_in_range(n1, n2)) {
            s = dot / (sqrtf(n1) * sqrtf(n2));
        } else {
            const CRow r = cos_reread<BF16>(pr, qr, a.Dc, lane);
            s = r.s;
            bad_row = bad_row || r.nonfinite;
        }
    }

    if (lane == 0) {
        float cv2 = 0.f, h2 = 0.f;
        const float Df = (float)a.D;
        const float mean = sh.c + sd / Df;   // of the scaled |x|
        if constexpr (kH1) {
            // cv2 holds the key KL = log D - H1, h2 holds H1.
            if (zero_row || !(mean > 0.f)) {   // all-zero row: H1 = 0
                cv2 = a.logD;
                h2 = 0.f;
            } else {
                const float rm1 = fmaf(sd / Df, sh.inv_c, sh.delta);   // r - 1
                const float r = 1.f + rm1;
                const float gr = Df * g2_shannon(rm1 * kInvLn2, r);
                // sum g(u_j) >= D g(r) (Jensen), with equality only when every
                // u_j is equal; for any other row the difference is at least
                // about n_probe / (n_probe + D) of the sum.  A difference
                // within the rounding of the sums ((D / 64 + 16) ulps) is an
                // exactly uniform row, whose KL is 0 at any magnitude (such
                // rows then tie exactly, as Eq. 3 makes them).
                const float num = sd2 - gr;
                const float thr = (Df * (1.f / kWave) + 16.f) * 0x1p-24f;
                const float dkl = fabsf(num) <= thr * (sd2 + gr) ? 0.f : kLn2 * num / r;
                cv2 = fmaxf(0.f, dkl / Df);
                h2 = a.logD - cv2;
            }
        } else if constexpr (kX) {
            const float m2 = fmaxf(0.f, fmaf(-sd, sd / Df, sd2));
            if (zero_row || !(mean > 0.f)) {   // all-zero row: H2 = 0, i.e. 1 + CV^2 = D
                cv2 = Df - 1.f;
                h2 = 0.f;
            } else {
                cv2 = (m2 / (mean * Df)) / mean;
                h2 = a.logD - log1pf(cv2);
            }
        }
        if (a.key_imp) a.key_imp[row] = cv2;
        if (a.key_s) a.key_s[row] = s;
        if (kX && a.out_h2) a.out_h2[row] = h2;
        if (kC && a.out_s) a.out_s[row] = s;
        if (a.nonfinite && bad_row) atomicAdd(a.nonfinite, 1u);
    }
}

// One wavefront per workgroup: the finest scheduling grain spreads rows evenly
// over the 256 CUs (measured 128 us vs 136 us with four-wavefront groups on
// 64 x 576 x 4096 bf16 rows).
//
// A wavefront issues up to four chunks of every tensor at once (kBurst), which
// hides the latency that bounds small launches (576 x 4096 bf16 rows 12.1 -> 9.0
// us a call against loads that waited for one another) and reaches HBM's rate in
// most large ones.  Where a launch lasts for many rounds of wavefronts, more bytes
// in flight than the round trip needs (about 27 KB a CU) only queue before the
// memory, and paced reads are faster: a wavefront keeps X's chunk, then X_pre's
// and X_post's in flight, and unused LDS limits the wavefronts of a CU.  A launch
// of few rounds must not be paced: a CU without its share of wavefronts, in the
// last round or with few rows at all, then waits for one chunk at a time.
//
// So the rule is one of rows (a round is 5120 of them with 20 wavefronts a CU),
// and of row sizes, below which a row's few chunks are paced by nothing.  us,
// burst against paced with that many wavefronts:
//   X and states, 20: 8 KB rows (bf16) 48828 of them 177.4 / 170.2, 36621 131.5 /
//     128.7, 24414 90.8 / 90.7; 6 KB 48828 133.4 / 129.4; 12 KB 32552 174.8 / 182.2;
//     3 KB 130208 181.8 / 176.0, 32552 46.9 / 48.5; 2 KB 195312 183.6 / 189.3; Shannon,
//     5 KB 58593 136.9 / 134.6, 4 KB 73242 134.1 / 135.9, 3 KB 97656 136.5 / 145.5.
//   16 wavefronts from 1.6 GB on, for rows of 7 KB: 262144 829.9 (20) / 819.4 (16),
//     8 KB 97656 336.9 / 335.1, fp32 12 KB 65104 342.8 / 335.3, 3 KB 130208 180.8 /
//     190.8; from 2 GB on with fewer rows too, 24414 fp32 rows of 32 KB 353.7 (burst)
//     / 343.6.  Shannon over bf16 rows has more to compute and stays at 20: 97656
//     341.5 (20) / 352.3 (16).
//   States alone, 28: 8 KB 146484 355.1 / 338.7, 36621 88.2 / 87.3, 18310 44.5 / 44.5,
//     9155 22.7 / 26.9.
//   X alone, all 32: 8 KB 146484 179.2 / 173.8, 73242 91.2 / 89.4, 36621 46.9 / 48.2;
//     Shannon, 3 KB 195312 185.9 / 167.2, 8 KB 36621 75.4 / 80.3.
//   X and states or states alone, 2 KB rows, all 32 (no pace but the chunk's own):
//     states 585937 362.7 / 340.0, 146484 87.0 / 87.6.
//   X and states of different widths, 28, from 1 GB on (columns that one of them
//     has alone are read one chunk at a time, which 20 wavefronts are too few for:
//     97656 rows of 4096 and 1024 bf16 181.6 in bursts, 190.4 with 20, 176.2 with 28):
//     1024 and 4096 bf16 130208 365 / 346, 32552 90.5 / 92.4; Shannon over bf16 rows
//     wider than the states stays in bursts (97656 of 4096 and 1024 240 / 239, 73242
//     of 4096 and 2048 196 / 200).
constexpr int64_t kManyRows = 35840;   // seven rounds

// LDS bytes a workgroup of a paced launch asks for (which set the wavefronts of a
// CU: 8 KB 20, 10 KB 16, 5.3 KB 28, none 32), or -1: not paced.
template <bool BF16, int MODE>
int paced_lds(int64_t rows, int64_t D, int64_t Dc)
{
    constexpr int kEB = Layout<BF16>::kEB;
    constexpr bool kX = (MODE & kScoreImp) != 0, kC = (MODE & kScoreSim) != 0, kH1 = (MODE & kScoreShannon) != 0;
    constexpr int k20 = 8192, k16 = 10240, k28 = 5440, k32 = 0;
    constexpr int64_t kKB = 1 << 10, kMB = 1 << 20;
    const int64_t row_bytes = (kX ? D : Dc) * kEB, total = rows * ((kX ? D : 0) + (kC ? 2 * Dc : 0)) * kEB;
    if (kX && kC && D != Dc) {
        const bool many = rows >= kManyRows && total >= 1000000000 && (D > Dc ? D : Dc) * kEB >= 4 * kKB;
        return many && !(kH1 && BF16 && D > Dc) ? k28 : -1;
    }
    if (!kC) {
        if (kH1) return rows >= 40960 && row_bytes >= 2 * kKB ? k32 : -1;
        return rows >= 49152 && row_bytes >= 6 * kKB && total >= 512 * kMB ? k32 : -1;
    }
    if (!kH1 && row_bytes >= 2 * kKB && row_bytes < 3 * kKB) return rows >= 150000 ? k32 : -1;
    if (!kX) return rows >= kManyRows && row_bytes >= 3 * kKB && total >= 512 * kMB ? k28 : -1;
    const bool wide = row_bytes >= 7 * kKB && !(kH1 && BF16);
    if (wide && total >= 2000000000 && rows >= 12000) return k16;
    if (rows < kManyRows || row_bytes < (kH1 ? 5 : 3) * kKB) return -1;
    return wide && total >= 1600000000 ? k16 : k20;
}

template <bool BF16, int MODE>
hipError_t launch_t(const ScoreArgs& a, hipStream_t s)
{
    if (a.rows <= 0) return hipSuccess;
    constexpr int V = Layout<BF16>::kV;
    constexpr bool kX = (MODE & kScoreImp) != 0, kC = (MODE & kScoreSim) != 0;
    const dim3 grid((unsigned)a.rows), block(kWave);
    const int lds = paced_lds<BF16, MODE>(a.rows, a.D, a.Dc);
    if ((kX && a.D % V) || (kC && a.Dc % V)) {
        hipLaunchKernelGGL((score_kernel<BF16, MODE, kOdd>), grid, block, 0, s, a);
    } else if (lds >= 0) {
        hipLaunchKernelGGL((score_kernel<BF16, MODE, kPaced>), grid, block, lds, s, a);
    } else {
        hipLaunchKernelGGL((score_kernel<BF16, MODE, kBurst>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

template <bool BF16>
hipError_t launch_m(const ScoreArgs& a, int mode, hipStream_t s)
{
    constexpr int I = kScoreImp, S = kScoreSim, H = kScoreShannon;
    switch (mode) {
    case I: return launch_t<BF16, I>(a, s);
    case S: return launch_t<BF16, S>(a, s);
    case I | S: return launch_t<BF16, I | S>(a, s);
    case I | H: return launch_t<BF16, I | H>(a, s);
    default: return launch_t<BF16, I | S | H>(a, s);
    }
}

}  // namespace

hipError_t launch_score(const ScoreArgs& a, bool bf16, int mode, hipStream_t s)
{
    const int base = mode & ~kScoreShannon;
    if (base != kScoreImp && base != kScoreSim && base != (kScoreImp | kScoreSim)) return hipErrorInvalidValue;
    if ((mode & kScoreShannon) && !(mode & kScoreImp)) mode &= ~kScoreShannon;
    return bf16 ? launch_m<true>(a, mode, s) : launch_m<false>(a, mode, s);
}

}  // namespace tr
