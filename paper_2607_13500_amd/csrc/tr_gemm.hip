// bf16 matrix-core GEMM for the steps around the path:
//   C[M, N] = A[M, K] . B[N, K]^T      (bf16 in, fp32 accumulation, bf16 out)
// with two optional fusions:
//   * row gather of A (A row m is A[rows[m]]): the projector GEMM applied to
//     the kept tokens straight from X, without materialising the gathered
//     copy (the step after the path: the kept tokens are projected);
//   * cosine epilogue: while the fp32 tile of C is in registers, per-row
//     partial sums of P.C, P.P and C.C against a second [M, N] matrix P.  With
//     C = x'' the output of the encoder MLP's second layer (W2 applied to the
//     hidden activations) and P = x' its input, these are Eq. (6)'s three sums,
//     so the Stage II score needs no further pass over X_pre or X_post.  The
//     sums use C as stored (rounded to bf16), so the score is Eq. (6) on the
//     x'' the caller receives, as an unfused scoring pass would compute it; a
//     row whose squared norms leave that pass's range is read again and scaled
//     as there (cos_finish_kernel).
//
// Two kernels for gfx950 (64-wide wavefronts, 32x32x16 bf16 MFMA), both with
// the same per-element MFMA sequence (k ascending in steps of 16), so they give
// bit-identical C:
//   * large: workgroup tile (64 MT) x 256 x 64 with MT = 4, 3 or 2 picked per
//     shape so the tiles fill the CUs in whole waves, operands straight from
//     global memory into LDS; described at the kernel.
//   * narrow (operands beyond 31-bit buffer offsets): workgroup tile 256 x 128
//     x 64 with 64-bit addresses, four wavefronts of 128 x 64, rows padded from
//     128 to 144 bytes for conflict-free fragment reads, the next k-tile
//     prefetched into registers (54 KB of LDS: two workgroups fit a CU).
// Both spread the output tiles over the XCDs (workgroup b runs on XCD b % 8)
// so that the workgroups sharing operand rows share an XCD's L2.
//
// MFMA operand layout (32x32x16 bf16, verified on the device): lane l holds
// A row l % 32 and B column l % 32, k = (l / 32) * 8 .. + 8; accumulator
// element v of lane l is C[(v / 4) * 8 + (l / 32) * 4 + v % 4][l % 32].
#include <cstdlib>
#include <type_traits>

#include "tr_internal.h"
#include "tr_row.h"
#include "tr_wave.h"

namespace tr {
namespace {

constexpr int kBM = 256, kBN = 128, kBK = 64;
constexpr int kThreads = 256;
constexpr int kRowBytes = 144;                       // 64 bf16 + 16 bytes of padding
constexpr int kLdsA = kBM * kRowBytes;               // 36864
constexpr int kLdsB = kBN * kRowBytes;               // 18432
constexpr int kLdsRed = 2 * kBM * 3 * 4;             // cosine partials of the two N-halves
constexpr int kXcds = 8;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }

// bf16 round-to-nearest-even of an fp32 value (NaN stays NaN), in hardware.
__device__ __forceinline__ uint16_t to_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// A partial sum of squares that came out as 0 although some of its elements are
// not (their products underflow): a value below every accepted norm in its
// place, so that only rows of zeros end with a norm of exactly 0.
__device__ __forceinline__ float mark_underflow(float sum, bool some) { return sum == 0.f && some ? 0x1p-126f : sum; }

template <bool GATHER, bool COS>
__global__ __launch_bounds__(kThreads, 2) void gemm_kernel(GemmArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* lA = smem;
    unsigned char* lB = smem + kLdsA;

    // ---- tile of this workgroup (XCD-aware order) --------------------------
    const int mt = (a.M + kBM - 1) / kBM, nt = a.N / kBN;
    const int tiles = mt * nt;
    const int per_xcd = (tiles + kXcds - 1) / kXcds;
    const int t = (int)(blockIdx.x % kXcds) * per_xcd + (int)(blockIdx.x / kXcds);
    if (t >= tiles) return;   // whole workgroup leaves together
    const int m0 = (t / nt) * kBM, n0 = (t % nt) * kBN;

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wm = w >> 1, wn = w & 1;   // 2 x 2 wavefront grid

    // ---- global -> register loads: thread owns 16-byte chunk (tid % 8) of
    // rows tid / 8 + 32 p.  A: 8 rows per thread, B: 4.
    const int ch = tid & 7, r0 = tid >> 3;
    // Rows outside the matrix (or gathered indices out of range) load row 0
    // and are zeroed when stored to LDS: the loads stay unconditional, so
    // nothing waits on them before the MFMAs of the current k-tile.
    const char* arow[8];
    uint32_t avalid = 0;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        const int m = m0 + r0 + 32 * p;
        int64_t src = -1;
        if (m < a.M) {
            src = m;
            if constexpr (GATHER) {
                const int32_t r = a.arows[m];
                src = (r >= 0 && r < a.arow_count) ? (int64_t)r : -1;
            }
        }
        if (src >= 0) avalid |= 1u << p;
        arow[p] = reinterpret_cast<const char*>(a.A) + (src >= 0 ? src : 0) * a.lda * 2 + ch * 16;
    }
    const char* brow[4];
#pragma unroll
    for (int p = 0; p < 4; ++p)
        brow[p] = reinterpret_cast<const char*>(a.B) + (int64_t)(n0 + r0 + 32 * p) * a.ldb * 2 + ch * 16;

    u32x4 ra[8], rb[4];
    auto load_tile = [&](int k0) {
#pragma unroll
        for (int p = 0; p < 8; ++p)
            ra[p] = *reinterpret_cast<const u32x4*>(arow[p] + (int64_t)k0 * 2);
#pragma unroll
        for (int p = 0; p < 4; ++p) rb[p] = *reinterpret_cast<const u32x4*>(brow[p] + (int64_t)k0 * 2);
    };
    auto store_tile = [&]() {
#pragma unroll
        for (int p = 0; p < 8; ++p)
            *reinterpret_cast<u32x4*>(lA + (r0 + 32 * p) * kRowBytes + ch * 16) =
                ((avalid >> p) & 1u) ? ra[p] : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int p = 0; p < 4; ++p)
            *reinterpret_cast<u32x4*>(lB + (r0 + 32 * p) * kRowBytes + ch * 16) = rb[p];
    };

    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // fragment addresses inside the LDS tiles
    const int frow = lane & 31, fk = (lane >> 5) * 16;   // byte offset of the lane's 8 k values
    const unsigned char* fa = lA + (wm * 128 + frow) * kRowBytes + fk;
    const unsigned char* fb = lB + (wn * 64 + frow) * kRowBytes + fk;

    const int KT = a.K / kBK;
    load_tile(0);
    store_tile();
    __syncthreads();
    for (int kt = 0; kt < KT; ++kt) {
        if (kt + 1 < KT) load_tile((kt + 1) * kBK);
#pragma unroll
        for (int kk = 0; kk < kBK / 16; ++kk) {
            bf16x8 fA[4], fB[2];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                fA[i] = *reinterpret_cast<const bf16x8*>(fa + i * 32 * kRowBytes + kk * 32);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                fB[j] = *reinterpret_cast<const bf16x8*>(fb + j * 32 * kRowBytes + kk * 32);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fA[i], fB[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
        if (kt + 1 < KT) {
            store_tile();
            __syncthreads();
        }
    }

    // ---- epilogue ---------------------------------------------------------
    const int half = lane >> 5;
    uint16_t* C = reinterpret_cast<uint16_t*>(a.C);
    float* red = reinterpret_cast<float*>(smem + kLdsA + kLdsB);   // [2][kBM][3]
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int rl = wm * 128 + i * 32 + (v >> 2) * 8 + half * 4 + (v & 3);   // row in the tile
            const int m = m0 + rl;
            const bool ok = m < a.M;
            float dot = 0.f, pp = 0.f, cc = 0.f;
            [[maybe_unused]] bool some_p = false, some_c = false;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int n = n0 + wn * 64 + j * 32 + (lane & 31);
                const uint16_t cb = to_bf16(acc[i][j][v]);
                const float c = bf16_lo(cb);   // the value stored
                [[maybe_unused]] float p = 0.f;
                if constexpr (COS)   // before C is stored, which may be P
                    if (ok) p = bf16_lo(reinterpret_cast<const uint16_t*>(a.P)[(int64_t)m * a.ldp + n]);
                if (ok) C[(int64_t)m * a.ldc + n] = cb;
                if constexpr (COS) {
                    dot = fmaf(p, c, dot);
                    pp = fmaf(p, p, pp);
                    cc = fmaf(c, c, cc);
                    some_p |= p != 0.f;
                    some_c |= c != 0.f;
                }
            }
            if constexpr (COS) {
                pp = mark_underflow(pp, some_p);
                cc = mark_underflow(cc, some_c);
                // sum over the 32 lanes of this half (same row): lane 31 / 63 ends with it
                dot = half_sum(dot);
                pp = half_sum(pp);
                cc = half_sum(cc);
                if ((lane & 31) == 31) {
                    float* r = red + ((size_t)wn * kBM + rl) * 3;
                    r[0] = dot;
                    r[1] = pp;
                    r[2] = cc;
                }
            }
        }
    }
    if constexpr (COS) {
        __syncthreads();
        // one thread per tile row: the two N-halves, then this tile's partials
        const int rl = tid;
        const int m = m0 + rl;
        if (m < a.M) {
            const float* r0p = red + (size_t)rl * 3;
            const float* r1p = red + ((size_t)kBM + rl) * 3;
            float* out = a.part + ((int64_t)m * a.part_cols + n0 / kBN) * 3;
            out[0] = r0p[0] + r1p[0];
            out[1] = r0p[1] + r1p[1];
            out[2] = r0p[2] + r1p[2];
        }
    }
}

// ---- tiles fed through LDS by LDS-destination loads -------------------------
constexpr uint32_t kBufWord3 = 0x00020000u;        // raw buffer resource, 32-bit elements
constexpr uint32_t kBadRow = 0x80000000u;          // a buffer offset past every resource
constexpr int kSlot = 16384;                       // 128 rows of one k-tile (64 bf16 each)

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(2)));   // 16 bytes at any element
typedef __attribute__((address_space(3))) unsigned char lds_t;
typedef __attribute__((address_space(3))) bf16x8 lds_frag;
typedef __attribute__((address_space(3))) bf16x4 lds_quad;
typedef __attribute__((address_space(3))) u32x4 lds_chunk;
typedef __attribute__((address_space(3))) float lds_f32;

// Buffer resource over `bytes` bytes at p (wave-uniform); loads past it read 0.
__device__ __forceinline__ u32x4 buffer_of(const void* p, int64_t bytes)
{
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    u32x4 r;
    r.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    r.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu));
    r.z = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)(bytes < (int64_t)kBadRow ? (uint32_t)bytes : kBadRow - 1u));
    r.w = kBufWord3;
    return r;
}

// 16 bytes a lane from the buffer straight into LDS at lds + 16 lane.  Written
// as an instruction (it has no register result) so that the compiler does not
// tie it to every later LDS read: the kernels below count the loads in flight
// themselves and wait for exactly those a barrier is about to publish.
__device__ __forceinline__ void load_lds(u32x4 r, uint32_t lds, uint32_t voff, uint32_t soff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(r), "s"(soff) : "memory", "m0");
}

// At most n of this wavefront's loads still in flight.
template <int n>
__device__ __forceinline__ void wait_loads()
{
    static_assert(n >= 0 && n < 64, "vmcnt is six bits");
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(n) : "memory");
}

// This wavefront's LDS reads have returned.
__device__ __forceinline__ void wait_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Workgroup barrier alone: no wait for memory, nothing scheduled across it.
__device__ __forceinline__ void barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
}

// Sum over each group of eight lanes, in every lane of the group.
__device__ __forceinline__ float sum8(float x)
{
    auto dpp = [](float v, auto ctrl) {
        return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(
            0, (int)__float_as_uint(v), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    x += dpp(x, std::integral_constant<int, 0xB1>{});    // lane ^ 1
    x += dpp(x, std::integral_constant<int, 0x4E>{});    // lane ^ 2
    x += dpp(x, std::integral_constant<int, 0x141>{});   // 7 - lane within the eight
    return x;
}

// Output tile of workgroup b: XCD b % 8 takes a contiguous run of tiles, and
// the run walks blocks of kTileRows tile rows column by column, so the tiles
// an XCD works on at once form a block of few rows and few columns and share
// both operands in its L2.  8192^3, 256 x 256 tiles: 837 -> 792 us against
// rows of tiles (the operands alone took 757 us to load there).
constexpr int kTileRows = 4;

__device__ __forceinline__ bool tile_of(int mt, int nt, int& tm, int& tn)
{
    const int tiles = mt * nt, per_xcd = (tiles + kXcds - 1) / kXcds;
    const int t = (int)(blockIdx.x % kXcds) * per_xcd + (int)(blockIdx.x / kXcds);
    if (t >= tiles) return false;
    const int group = t / (kTileRows * nt), in = t % (kTileRows * nt);
    const int rows = mt - group * kTileRows < kTileRows ? mt - group * kTileRows : kTileRows;
    tm = group * kTileRows + in % rows;
    tn = in / rows;
    return true;
}

// Epilogue of a wavefront that holds a (32 RB) x (32 CB) block of C with its
// first element at (m, n).  The MFMA operands are exchanged (B's fragment
// first), so lane l holds row l % 32 of each 32 x 32 block and, in v =
// 4 q .. 4 q + 3, the four consecutive columns 8 q + 4 (l / 32): they are
// rounded to bf16 (v_cvt_pk_bf16_f32, nearest even), put into the
// wavefront's own LDS rows (64 CB bytes, 16-byte chunks swizzled by row) and
// read back as 16-byte pieces of rows, which leave as full cache lines.
// Rounding in integer code and storing each value by itself took 4100
// instructions a wavefront and 15 us of a 115 us 4096^3 product.
// With COS the same pieces give the row sums P.C, P.P and C.C over the
// block's columns (the values as stored), left in red[row][3].
template <int RB, int CB, bool COS>
__device__ __forceinline__ void finish_block(const GemmArgs& a, const f32x16 (&acc)[RB][CB], lds_t* own, int m,
                                             int n, lds_f32* red)
{
    constexpr int kChunks = 4 * CB, kRowsStep = kWave / kChunks, kSteps = 32 * RB / kRowsStep;
    constexpr int kRowB = 64 * CB;
    const int lane = threadIdx.x & 63, l31 = lane & 31, half = lane >> 5;
    const int c = lane % kChunks, r0 = lane / kChunks;
    [[maybe_unused]] u32x4 p[COS ? kSteps : 1];
    if constexpr (COS) {
        const uint16_t* P = reinterpret_cast<const uint16_t*>(a.P) + n + c * 8;
#pragma unroll
        for (int g = 0; g < kSteps; ++g) {
            const int row = m + g * kRowsStep + r0;
            p[g] = row < a.M ? *reinterpret_cast<const u32x4_any*>(P + (int64_t)row * a.ldp) : u32x4{0u, 0u, 0u, 0u};
        }
    }
    auto at = [&](int r, int ch) { return own + r * kRowB + ((ch ^ ((CB == 2 ? r >> 1 : r >> 2) & (kChunks - 1))) * 16); };
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 x = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                *(lds_quad*)(at(i * 32 + l31, j * 4 + q) + half * 8) = __builtin_convertvector(x, bf16x4);
            }
    uint16_t* C = reinterpret_cast<uint16_t*>(a.C) + n + c * 8;
#pragma unroll
    for (int g = 0; g < kSteps; ++g) {
        const int r = g * kRowsStep + r0;
        const u32x4 v = *(const lds_chunk*)at(r, c);
        if (m + r < a.M) *reinterpret_cast<u32x4_any*>(C + (int64_t)(m + r) * a.ldc) = v;
        if constexpr (COS) {
            static_assert(!COS || kChunks == 8, "a row's sums are over eight lanes");
            float d = 0.f, pp = 0.f, cc = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                d = dot2(p[g][k], v[k], d);
                pp = dot2(p[g][k], p[g][k], pp);
                cc = dot2(v[k], v[k], cc);
            }
            auto some = [](u32x4 x) { return ((x[0] | x[1] | x[2] | x[3]) & 0x7fff7fffu) != 0u; };   // not all +-0
            pp = mark_underflow(pp, some(p[g]));
            cc = mark_underflow(cc, some(v));
            d = sum8(d);
            pp = sum8(pp);
            cc = sum8(cc);
            if (c == 0) {
                red[r * 3] = d;
                red[r * 3 + 1] = pp;
                red[r * 3 + 2] = cc;
            }
        }
    }
}

// The tile's partial sums from those of its WN column blocks, in their order.
template <int ROWS, int WN, int THREADS>
__device__ __forceinline__ void finish_sums(const GemmArgs& a, const lds_f32* red, int m0, int tn)
{
    for (int r = threadIdx.x; r < ROWS; r += THREADS) {
        if (m0 + r >= a.M) continue;
        float s[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < WN; ++q)
#pragma unroll
            for (int k = 0; k < 3; ++k) s[k] += red[(q * ROWS + r) * 3 + k];
        float* out = a.part + ((int64_t)(m0 + r) * a.part_cols + tn) * 3;
#pragma unroll
        for (int k = 0; k < 3; ++k) out[k] = s[k];
    }
}

// ---- large tiles: (64 MT) x 256, eight wavefronts in two alternating groups --
//
// Wavefront (wm, wn) of the 2 x 4 grid owns (32 MT) x 64 of C; the two
// wavefronts of a SIMD are of different wm.  A k-tile (64 of K) lies in LDS
// as four parts, each read whole in one phase: A0 (the wavefronts' first 64
// rows), A1 (the rest), B0 and B1 (their first and second 32 columns); two
// k-tiles are held.  Each phase of a wavefront is a memory part (LDS reads of
// the fragments it needs next, LDS-destination loads into the part that the
// phase before has freed) and an MFMA part (8 MFMAs, 256 cycles), separated
// by barriers; the wm = 1 wavefronts run one barrier behind, so each SIMD's
// matrix pipe always has one wavefront in its MFMA part while the other
// reads (without the offset: 106 -> 123 us at 4096^3).  A part is refilled as
// soon as it is free, so its loads have nearly two k-tiles to arrive and no
// wait ever drains the queue.
//
// Bound by the matrix pipes and the clock that the chip holds under them: at
// 4096^3 they are busy for 131 of the launch's 184 thousand cycles, at 1.7 of 2.4
// GHz; the LDS is busy for 52 thousand.  105 us (a two-stage loop that waits for
// all loads before each k-tile: 114 us; the library's kernel: 90 us).  Barrier
// counts are equal in every wavefront: each runs the same phases and one extra
// barrier (wm = 1 before, wm = 0 after).
constexpr int kPBN = 256, kPThreads = 512, kPBuf = 4 * kSlot;
constexpr int kOffA1 = kSlot, kOffB0 = 2 * kSlot, kOffB1 = 3 * kSlot;

template <int MT, bool GATHER, bool COS>
__global__ __launch_bounds__(kPThreads, 1) void gemm_large_kernel(GemmArgs a)
{
    static_assert(MT >= 2 && MT <= 4, "A1 holds MT - 2 blocks of 32 rows per wavefront");
    constexpr int BM = 64 * MT;
    constexpr int kA1 = MT - 2;          // LDS-destination loads of A1 per wavefront (A0, B0, B1: 2 each)
    __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * kPBuf];
    __shared__ float red_[COS ? 4 * BM * 3 : 1];
    lds_t* const sm = (lds_t*)smem;
    const uint32_t sbase = (uint32_t)(uintptr_t)sm;

    int tm, tn;
    if (!tile_of((a.M + BM - 1) / BM, (a.N + kPBN - 1) / kPBN, tm, tn)) return;   // whole workgroup
    const int m0 = tm * BM, n0 = tn * kPBN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w >> 2, wn = w & 3;

    // ---- global -> LDS.  Rows of 128 bytes; lane l of wavefront w fills
    // physical chunk l % 8 of row 64 j + 8 w + l / 8 of a part, which holds
    // logical chunk (l % 8) ^ ((row / 2) % 8).  Rows past A or B, and gathered
    // rows out of range, lie past the resource and read as zeros.
    const uint16_t* A = reinterpret_cast<const uint16_t*>(a.A);
    const uint16_t* B = reinterpret_cast<const uint16_t*>(a.B);
    const u32x4 ra = GATHER ? buffer_of(A, a.arow_count * a.lda * 2)
                            : buffer_of(A + (int64_t)m0 * a.lda, (int64_t)(a.M - m0) * a.lda * 2);
    const u32x4 rb = buffer_of(B + (int64_t)n0 * a.ldb, (int64_t)(a.N - n0) * a.ldb * 2);
    uint32_t oa0[2], oa1[2], ob[2][2];
    {
        const int row = w * 8 + (lane >> 3);
        const uint32_t c = (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) * 16);
        auto a_off = [&](int r) -> uint32_t {   // r: row of the tile
            if constexpr (GATHER) {
                const int g = m0 + r < a.M ? a.arows[m0 + r] : -1;
                return (g >= 0 && g < a.arow_count) ? (uint32_t)((int64_t)g * a.lda * 2) + c : kBadRow;
            } else {
                return (uint32_t)(r * a.lda * 2) + c;
            }
        };
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            oa0[j] = a_off(j * 32 * MT + row);
            if constexpr (MT == 4) oa1[j] = a_off(j * 32 * MT + 64 + row);
#pragma unroll
            for (int h = 0; h < 2; ++h)
                ob[h][j] = (uint32_t)(((2 * j + (row >> 5)) * 64 + h * 32 + (row & 31)) * a.ldb * 2) + c;
        }
        if constexpr (MT == 3) oa1[0] = a_off((row >> 5) * 96 + 64 + (row & 31));
    }
    const uint32_t dst = sbase + (uint32_t)w * 1024;
    auto buf_of = [](int kt) { return (uint32_t)(kt & 1) * kPBuf; };
    auto load_a0 = [&](int kt) {
#pragma unroll
        for (int j = 0; j < 2; ++j) load_lds(ra, dst + buf_of(kt) + j * 8192, oa0[j], (uint32_t)kt * 128);
    };
    auto load_a1 = [&](int kt) {
#pragma unroll
        for (int j = 0; j < kA1; ++j) load_lds(ra, dst + buf_of(kt) + kOffA1 + j * 8192, oa1[j], (uint32_t)kt * 128);
    };
    auto load_b = [&](int h, int kt) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
            load_lds(rb, dst + buf_of(kt) + (h ? kOffB1 : kOffB0) + j * 8192, ob[h][j], (uint32_t)kt * 128);
    };

    // ---- fragment reads: lane l reads row l % 32 of a 32-row block, logical
    // chunk 2 kk + l / 32
    const int l31 = lane & 31, half = lane >> 5;
    uint32_t fa[4], fb[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const uint32_t cb = (uint32_t)(((2 * kk + half) ^ ((l31 >> 1) & 7)) * 16);
        fa[kk] = (uint32_t)l31 * 128 + cb;
        fb[kk] = (uint32_t)(wn * 32 + l31) * 128 + cb;
    }
    f32x16 acc[MT][2];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    // Fragments of A0, of A1 (in A0's place when the phases allow it) and of
    // both column blocks.
    bf16x8 fA[MT == 3 ? 3 : 2][4], fB[2][4];
    auto read_a0 = [&](int kt) {
        const lds_t* p = sm + (buf_of(kt) + (uint32_t)wm * 8192);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int i = 0; i < 2; ++i) fA[i][kk] = *(const lds_frag*)(p + fa[kk] + i * 4096);
    };
    auto read_a1 = [&](int kt) {
        const lds_t* p = sm + (buf_of(kt) + kOffA1 + (uint32_t)(wm * 4096 * kA1));
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int i = 0; i < kA1; ++i) fA[MT == 3 ? 2 : i][kk] = *(const lds_frag*)(p + fa[kk] + i * 4096);
    };
    auto read_b = [&](int h, int kt) {
        const lds_t* p = sm + (buf_of(kt) + (h ? kOffB1 : kOffB0));
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) fB[h][kk] = *(const lds_frag*)(p + fb[kk]);
    };
    // Blocks i0 .. i0 + n - 1 of the wavefront's rows (fragments from f0 on)
    // times column blocks j0 .. j1, between barriers.
    auto mma = [&](int i0, int n, int f0, int j0, int j1) {
        wait_reads();
        barrier();
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int i = 0; i < n; ++i)
#pragma unroll
                for (int j = j0; j <= j1; ++j)
                    acc[i0 + i][j] =
                        __builtin_amdgcn_mfma_f32_32x32x16_bf16(fB[j][kk], fA[f0 + i][kk], acc[i0 + i][j], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
        barrier();
    };

    // One k-tile.  Tail 0: kt + 2 exists; 1: kt is the last but one; 2: the
    // last.  Each wait leaves in flight exactly the loads issued after those
    // that the next phase reads; the barriers in between publish them.
    const int KT = a.K / kBK;
    auto step = [&](int kt, auto tail) {
        constexpr int T = decltype(tail)::value;
        constexpr bool more = T == 0, next = T < 2;
        if constexpr (MT == 4) {
            read_a0(kt);
            if constexpr (more) load_b(0, kt + 2);
            wait_loads<more ? 12 : next ? 10 : 2>();   // B1
            mma(0, 2, 0, 0, 0);
            read_b(1, kt);
            if constexpr (more) load_a0(kt + 2);
            wait_loads<more ? 12 : next ? 8 : 0>();    // A1
            mma(0, 2, 0, 1, 1);
            read_a1(kt);
            if constexpr (more) load_b(1, kt + 2);
            if constexpr (next) wait_loads<more ? 12 : 6>();   // B0 of kt + 1
            mma(2, 2, 0, 0, 0);
            if constexpr (next) read_b(0, kt + 1);
            if constexpr (more) load_a1(kt + 2);
            if constexpr (next) wait_loads<more ? 12 : 4>();   // A0 of kt + 1
            mma(2, 2, 0, 1, 1);
        } else if constexpr (MT == 3) {
            read_a0(kt);
            if constexpr (more) load_b(0, kt + 2);
            wait_loads<more ? 9 : next ? 7 : 0>();     // A1, B1
            mma(0, 2, 0, 0, 0);
            read_a1(kt);
            read_b(1, kt);
            if constexpr (more) load_a0(kt + 2);
            if constexpr (next) wait_loads<more ? 9 : 5>();    // B0 of kt + 1
            mma(2, 1, 2, 0, 1);
            if constexpr (next) read_b(0, kt + 1);
            if constexpr (more) {
                load_a1(kt + 2);
                load_b(1, kt + 2);
            }
            if constexpr (next) wait_loads<more ? 10 : 3>();   // A0 of kt + 1
            mma(0, 2, 0, 1, 1);
        } else {
            read_a0(kt);
            if constexpr (next) load_b(1, kt + 1);
            if constexpr (more) load_b(0, kt + 2);
            wait_loads<more ? 6 : next ? 4 : 0>();     // B1, B0 of kt + 1
            mma(0, 2, 0, 0, 0);
            read_b(1, kt);
            if constexpr (next) read_b(0, kt + 1);
            if constexpr (more) load_a0(kt + 2);
            if constexpr (next) wait_loads<more ? 6 : 2>();    // A0 of kt + 1
            mma(0, 2, 0, 1, 1);
        }
    };

    // The first two k-tiles, in the order in which the steps count them (MT =
    // 2 holds B1 for one phase less and loads it one k-tile ahead).
    load_b(0, 0);
    load_a0(0);
    load_b(1, 0);
    load_a1(0);
    if (KT > 1) {
        load_b(0, 1);
        load_a0(1);
        if constexpr (MT > 2) {
            load_b(1, 1);
            load_a1(1);
        }
        wait_loads<MT == 4 ? 12 : MT == 3 ? 10 : 6>();   // B0, A0 of the first
    } else {
        wait_loads<MT == 4 ? 4 : MT == 3 ? 3 : 2>();
    }
    barrier();
    read_b(0, 0);
    wait_reads();   // the first step refills B0
    barrier();
    if (wm == 1) barrier();
    int kt = 0;
    for (; kt + 2 < KT; ++kt) step(kt, std::integral_constant<int, 0>{});
    if (KT > 1) step(kt++, std::integral_constant<int, 1>{});
    step(kt, std::integral_constant<int, 2>{});
    if (wm == 0) barrier();

    // Every wavefront has read its last fragments: the buffers are free.
    lds_t* own = sm + w * (32 * MT * 128);
    lds_f32* red = (lds_f32*)red_;
    const int n = n0 + wn * 64;
    if (n < a.N)   // N is a multiple of 128: whole wavefronts lie past it
        finish_block<MT, 2, COS>(a, acc, own, m0 + wm * 32 * MT, n, red + (wn * BM + wm * 32 * MT) * 3);
    if constexpr (COS) {
        if (n >= a.N)
            for (int r = lane; r < 32 * MT * 3; r += kWave) red[(wn * BM + wm * 32 * MT) * 3 + r] = 0.f;
        wait_reads();
        barrier();
        finish_sums<BM, 4, kPThreads>(a, red, m0, tn);
    }
}

// s = dot / (|P| |C|) from the per-tile partials, summed in tile order, with the
// scoring kernel's reading of its sums: a zero vector gives s = 0, and a row
// whose squared norms leave the accepted range (states of magnitude 2^-75 to
// 2^-30, whose products underflow in part, or beyond 2^63) is read again by the
// wavefront, each vector scaled by its own maximum.  A wavefront takes few rows
// because it reads them again one by one.  Without a.P (C was stored over P) such
// a row keeps the cosine of its sums as they are, or 0 where a squared norm is so
// small that mark_underflow may have made it.
constexpr int kFinishRows = 16;   // rows of a wavefront

__global__ __launch_bounds__(256) void cos_finish_kernel(GemmArgs a, int cols)
{
    const int lane = threadIdx.x & 63;
    const int r0 = ((int)blockIdx.x * (256 / kWave) + (int)(threadIdx.x / kWave)) * kFinishRows;
    const int m = r0 + lane;
    float v = 0.f;
    bool again = false;
    if (lane < kFinishRows && m < a.M) {
        const float* p = a.part + (int64_t)m * a.part_cols * 3;
        float dot = 0.f, n1 = 0.f, n2 = 0.f;
        for (int c = 0; c < cols; ++c) {
            dot += p[3 * c];
            n1 += p[3 * c + 1];
            n2 += p[3 * c + 2];
        }
        if (cos_in_range(n1, n2) || (!a.P && n1 >= 0x1p-100f && n2 >= 0x1p-100f)) v = dot / (sqrtf(n1) * sqrtf(n2));
        else again = a.P && n1 != 0.f && n2 != 0.f;
    }
    for (uint64_t left = __ballot(again); left; left &= left - 1) {
        const int l = __ffsll((long long)left) - 1;
        const float s = cos_reread<true>(reinterpret_cast<const char*>(a.P) + (int64_t)(r0 + l) * a.ldp * 2,
                                         reinterpret_cast<const char*>(a.C) + (int64_t)(r0 + l) * a.ldc * 2, a.N,
                                         lane).s;
        if (lane == l) v = s;
    }
    if (lane < kFinishRows && m < a.M) a.s_out[m] = v;
}

// The large kernel takes every shape whose buffer offsets (rows of a tile, or
// all of A's rows when they are gathered) fit 31 bits: at N % 256 = 128 and K %
// 128 = 64 too it is the faster one (3001 x 1664 x 4160: 45 against 93 us).
bool use_large(const GemmArgs& a)
{
    const int64_t lim = (int64_t)kBadRow;
    if ((int64_t)kBM * a.lda * 2 >= lim || (int64_t)kPBN * a.ldb * 2 >= lim) return false;
    return !a.arows || a.arow_count * a.lda * 2 < lim;
}

int g_cus = 256;         // compute units of the device (set by gemm_prepare)
int g_force_mt = 0;      // tile height override: 0 = model, else 2, 3 or 4

// Tile height of the large kernel (MFMA tiles per wavefront along M): the one
// with the least modelled time, (tile waves over the CUs) x (rows per tile),
// where shorter tiles pay for their higher LDS traffic per MFMA.  Rates on
// shapes that fill the CUs, as 256 : 192 : 128 rows: 1340 : 1225 : 1180
// TFLOP/s (4096^3 and 36864 x 1024 x 4096), so 9 % and 14 % more per row.
int large_mt(int M, int N)
{
    if (g_force_mt) return g_force_mt;
    const double cost_per_row[5] = {0, 0, 1.14, 1.09, 1.0};
    int best = 4;
    double best_t = 0;
    for (int mtw = 4; mtw >= 2; --mtw) {
        const int64_t tiles = (int64_t)((M + 64 * mtw - 1) / (64 * mtw)) * ((N + kPBN - 1) / kPBN);
        const int64_t waves = (tiles + g_cus - 1) / g_cus;
        const double t = (double)waves * mtw * cost_per_row[mtw];
        if (mtw == 4 || t < best_t) {
            best = mtw;
            best_t = t;
        }
    }
    return best;
}

void launch_large(const GemmArgs& a, int mtw, bool gather, bool cos, int grid, hipStream_t s)
{
    const dim3 g(grid), b(kPThreads);
    if (mtw == 4) {
        if (gather)
            hipLaunchKernelGGL((gemm_large_kernel<4, true, false>), g, b, 0, s, a);
        else if (cos)
            hipLaunchKernelGGL((gemm_large_kernel<4, false, true>), g, b, 0, s, a);
        else
            hipLaunchKernelGGL((gemm_large_kernel<4, false, false>), g, b, 0, s, a);
    } else if (mtw == 3) {
        if (gather)
            hipLaunchKernelGGL((gemm_large_kernel<3, true, false>), g, b, 0, s, a);
        else if (cos)
            hipLaunchKernelGGL((gemm_large_kernel<3, false, true>), g, b, 0, s, a);
        else
            hipLaunchKernelGGL((gemm_large_kernel<3, false, false>), g, b, 0, s, a);
    } else {
        if (gather)
            hipLaunchKernelGGL((gemm_large_kernel<2, true, false>), g, b, 0, s, a);
        else if (cos)
            hipLaunchKernelGGL((gemm_large_kernel<2, false, true>), g, b, 0, s, a);
        else
            hipLaunchKernelGGL((gemm_large_kernel<2, false, false>), g, b, 0, s, a);
    }
}

}  // namespace

// capacity (row stride of the partials): the narrow kernel's column count
int gemm_part_cols(int N) { return N / kBN; }

bool gemm_shape_ok(int M, int N, int K)
{
    if (M < 0 || N <= 0 || K <= 0 || N % kBN || K % kBK) return false;
    // output tiles (and the grid, rounded up to the XCD count) fit an int
    const int64_t tiles = (int64_t)((M + (int64_t)kBM - 1) / kBM) * (N / kBN);
    return tiles <= (int64_t)INT32_MAX - kXcds;
}

hipError_t gemm_prepare()
{
    hipError_t e;
    int dev = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&g_cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    // TR_GEMM_TILE_ROWS = 128, 192 or 256 pins the large kernel's tile height
    // (tuning and tests); anything else leaves the choice to the model.
    const char* env = getenv("TR_GEMM_TILE_ROWS");
    const int rows = env ? atoi(env) : 0;
    g_force_mt = (rows == 128 || rows == 192 || rows == 256) ? rows / 64 : 0;
    const int lds = kLdsA + kLdsB + kLdsRed;
    if ((e = hipFuncSetAttribute((const void*)gemm_kernel<false, false>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds)) != hipSuccess) return e;
    if ((e = hipFuncSetAttribute((const void*)gemm_kernel<true, false>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds)) != hipSuccess) return e;
    return hipFuncSetAttribute((const void*)gemm_kernel<false, true>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, lds);
}

hipError_t launch_gemm(const GemmArgs& a, hipStream_t s)
{
    if (a.M == 0) return hipSuccess;
    const bool gather = a.arows != nullptr, cos = a.P != nullptr;
    if (gather && cos) return hipErrorInvalidValue;
    const bool large = use_large(a);
    const int mtw = large ? large_mt(a.M, a.N) : 4;
    const int bm = large ? 64 * mtw : kBM, bn = large ? kPBN : kBN;
    const int tiles = ((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn);
    const int grid = ((tiles + kXcds - 1) / kXcds) * kXcds;
    if (large) {
        launch_large(a, mtw, gather, cos, grid, s);
    } else {
        const size_t lds = kLdsA + kLdsB + (cos ? kLdsRed : 0);
        if (gather)
            hipLaunchKernelGGL((gemm_kernel<true, false>), dim3(grid), dim3(kThreads), lds, s, a);
        else if (cos)
            hipLaunchKernelGGL((gemm_kernel<false, true>), dim3(grid), dim3(kThreads), lds, s, a);
        else
            hipLaunchKernelGGL((gemm_kernel<false, false>), dim3(grid), dim3(kThreads), lds, s, a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !cos) return e;
    GemmArgs f = a;
    const char *p = static_cast<const char*>(a.P), *c = static_cast<const char*>(a.C);
    if (p < c + (int64_t)a.M * a.ldc * 2 && c < p + (int64_t)a.M * a.ldp * 2) f.P = nullptr;   // C lies over P
    constexpr int kRows = kFinishRows * (256 / kWave);
    hipLaunchKernelGGL(cos_finish_kernel, dim3((unsigned)(((int64_t)a.M + kRows - 1) / kRows)), dim3(256), 0, s, f,
                       (a.N + bn - 1) / bn);
    return hipGetLastError();
}

}  // namespace tr
