// Gather of the kept rows: out[r, :] = X[rows[r], :], byte for byte.
// A row is cut into pieces of 16 bytes, wherever it starts (the 16-byte accesses
// take any byte address); its last piece is its last 16 bytes, which overlap the
// piece before where the row is no multiple of 16 (both write the same bytes
// there).  Rows below 16 bytes, and some narrow ones (by_elements), go element by
// element.  A wavefront moves a row in columns of 64 pieces and issues the loads
// of exactly the columns the row has, up to eight, before its stores: loads past
// the row's end are not free, not even all of one address (selection and gather
// of 117,000 rows of 256 bytes in eight columns 53.7 us, in one 29.5).  Rows of at
// most 8 KiB go two to a wavefront, the second row's loads in flight while the
// first is stored (64 x 576 x 4096 bf16 step: 150.4 -> 148.8 us; four rows to a
// wavefront: 151.6 us); longer rows take one wavefront each.  Loads and stores
// are non-temporal: nothing is reused (non-temporal stores measured 8.6 vs 11.2 us
// for 4096 rows of 8 KiB).
#include "tr_internal.h"

namespace tr {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(2)));

// Columns j0 / 64 .. j0 / 64 + COLS - 1 of a row; END: the last of them is the
// row's last, which may be partial.
template <int COLS, bool END>
__device__ __forceinline__ void load_columns(const char* row, int j0, int pieces, int last, u32x4 (&v)[COLS])
{
#pragma unroll
    for (int u = 0; u < COLS; ++u) {
        const int j = j0 + kWave * u;
        const bool edge = END && u == COLS - 1;
        if (!edge || j < pieces)
            v[u] = __builtin_nontemporal_load(
                reinterpret_cast<const u32x4_any*>(row + (edge ? min(j * 16, last) : j * 16)));
    }
}

// PACED: one store of the wavefront in flight.
template <int COLS, bool END, bool PACED = false>
__device__ __forceinline__ void store_columns(char* row, int j0, int pieces, int last, const u32x4 (&v)[COLS])
{
#pragma unroll
    for (int u = 0; u < COLS; ++u) {
        const int j = j0 + kWave * u;
        const bool edge = END && u == COLS - 1;
        if constexpr (PACED) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (!edge || j < pieces)
            __builtin_nontemporal_store(v[u], reinterpret_cast<u32x4_any*>(row + (edge ? min(j * 16, last) : j * 16)));
    }
}

// The row's last columns, C of them (1 <= C <= COLS).
template <int COLS>
__device__ __forceinline__ void copy_end(const char* s, char* d, int j0, int pieces, int last, int c)
{
    if constexpr (COLS > 1) {
        if (c < COLS) return copy_end<COLS - 1>(s, d, j0, pieces, last, c);
    }
    u32x4 v[COLS];
    load_columns<COLS, true>(s, j0, pieces, last, v);
    store_columns<COLS, true>(d, j0, pieces, last, v);
}

template <int COLS>
__global__ __launch_bounds__(256) void gather_vec_kernel(const char* __restrict__ X, char* __restrict__ out,
                                                          const int32_t* __restrict__ rows,
                                                          int64_t nout, int64_t nrows, int64_t row_bytes)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t r = (int64_t)blockIdx.x * (blockDim.x / kWave) + (threadIdx.x / kWave);
    if (r >= nout) return;
    if (rows[r] < 0 || rows[r] >= nrows) return;   // memory safety against a bad index
    const char* s = X + (int64_t)rows[r] * row_bytes;
    char* d = out + r * row_bytes;
    const int pieces = (int)((row_bytes + 15) / 16), last = (int)row_bytes - 16;   // rows stay below 2 GB
    int c0 = 0;
    for (; pieces - c0 > kWave * COLS; c0 += kWave * COLS) {
        u32x4 v[COLS];
        load_columns<COLS, false>(s, c0 + lane, pieces, last, v);
        store_columns<COLS, false>(d, c0 + lane, pieces, last, v);
    }
    copy_end<COLS>(s, d, c0 + lane, pieces, last, (pieces - c0 + kWave - 1) / kWave);
}

// Rows of COLS columns, RPW consecutive output rows per wavefront: the loads
// of row k + 1 are in flight while row k is stored.
template <int COLS, int RPW, bool PACED>
__global__ __launch_bounds__(256) void gather_pipe_kernel(const char* __restrict__ X, char* __restrict__ out,
                                                           const int32_t* __restrict__ rows,
                                                           int64_t nout, int64_t nrows, int64_t row_bytes)
{
    const int pieces = (int)((row_bytes + 15) / 16), last = (int)row_bytes - 16;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t r0 = ((int64_t)blockIdx.x * (blockDim.x / kWave) + (threadIdx.x / kWave)) * RPW;
    if (r0 >= nout) return;
    // The source rows first: an index read between the copies would wait for
    // every load before it.
    int64_t src[RPW];
#pragma unroll
    for (int k = 0; k < RPW; ++k) src[k] = rows[r0 + k < nout ? r0 + k : r0];
    u32x4 v[2][COLS];
    auto ok = [&](int k) { return r0 + k < nout && src[k] >= 0 && src[k] < nrows; };   // memory safety against a bad index
    auto load = [&](int k) {
        load_columns<COLS, true>(X + (ok(k) ? src[k] : 0) * row_bytes, lane, pieces, last, v[k & 1]);
    };
    load(0);
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
        if (k + 1 < RPW) load(k + 1);
        if (ok(k)) store_columns<COLS, true, PACED>(out + (r0 + k) * row_bytes, lane, pieces, last, v[k & 1]);
    }
}

// One launch of gather_pipe_kernel with the rows' number of columns.
template <int COLS, int RPW, bool PACED>
void launch_pipe(int cols, dim3 grid, dim3 block, hipStream_t s, const char* X, char* out, const int32_t* rows,
                 int64_t nout, int64_t nrows, int64_t row_bytes)
{
    if constexpr (COLS > 1) {
        if (cols < COLS) {
            launch_pipe<COLS - 1, RPW, PACED>(cols, grid, block, s, X, out, rows, nout, nrows, row_bytes);
            return;
        }
    }
    hipLaunchKernelGGL((gather_pipe_kernel<COLS, RPW, PACED>), grid, block, 0, s, X, out, rows, nout, nrows, row_bytes);
}

template <typename E>
__global__ __launch_bounds__(256) void gather_elem_kernel(const E* __restrict__ X, E* __restrict__ out,
                                                          const int32_t* __restrict__ rows,
                                                          int64_t nout, int64_t nrows, int64_t elems_per_row)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t r = (int64_t)blockIdx.x * (blockDim.x / kWave) + (threadIdx.x / kWave);
    if (r >= nout) return;
    if (rows[r] < 0 || rows[r] >= nrows) return;   // memory safety against a bad index
    const E* s = X + (int64_t)rows[r] * elems_per_row;
    E* d = out + r * elems_per_row;
    for (int64_t j = lane; j < elems_per_row; j += kWave) d[j] = s[j];
}

// Whether a wavefront stores one column at a time.  Copies that the L2s (32 MB)
// or little more hold run faster so, at rows of some columns: stores in bursts
// get in the way of the loads.  Selection and gather of half of the rows, bursts ->
// one at a time: 4 KB rows 20 MB 16.1 -> 14.7 us, 29 MB 18.4 -> 17.1, 44 MB 22.9 ->
// 21.5, 69 MB 31.0 -> 30.6, 99 MB 41.5 -> 43.8; 8 KB rows 29 MB 17.7 -> 16.9, 69 MB
// 31.6 -> 30.4, 138 MB 54.2 -> 57.6; 2 KB rows 30 MB 18.8 -> 18.3, 45 MB 23.5 -> 24.6;
// 1 KB rows 20 MB 16.1 -> 15.9, 100 MB 42.6 -> 43.8.
bool paced_copy(int64_t bytes, int64_t row_bytes)
{
    return row_bytes >= 2048 && bytes < (row_bytes >= 4096 ? 80 : 36) * (int64_t)1000000;
}

// Whether rows that are no multiple of 16 bytes go element by element: an
// unaligned 16-byte store of a few lanes costs more than the row's elements from
// one or two steps of the wavefront, until the copy leaves the caches (pieces
// against elements: 66-byte rows 45 MB 120.7 us against 110.6, 252-byte fp32 rows
// 45 MB 42.3 against 37.8, 140 MB 118 against 142; 516-byte fp32 rows 10 MB 14.6
// against 14.0, 45 MB 30.3 against 31.6).
bool by_elements(int64_t bytes, int64_t row_bytes, int elem_bytes)
{
    if (row_bytes < 16) return true;
    const int64_t n = row_bytes / elem_bytes;
    return row_bytes % 16 && ((n <= kWave && bytes < 90000000) || (n <= 160 && bytes < 20000000));
}

}  // namespace

hipError_t launch_gather(const void* X, void* out, const int32_t* rows, int64_t nout, int64_t nrows,
                         int64_t row_bytes, int elem_bytes, hipStream_t s)
{
    if (nout <= 0) return hipSuccess;
    constexpr int kThreads = 256;
    const int64_t blocks = (nout + kThreads / kWave - 1) / (kThreads / kWave);
    constexpr int kCols = 8, kRowsPerWave = 2;
    const char* src = static_cast<const char*>(X);
    char* dst = static_cast<char*>(out);
    const int64_t bytes = nout * row_bytes;
    const bool elements = by_elements(bytes, row_bytes, elem_bytes);
    if (!elements && row_bytes <= 16 * kWave * kCols) {
        const int64_t waves = (nout + kRowsPerWave - 1) / kRowsPerWave;
        const int64_t pb = (waves + kThreads / kWave - 1) / (kThreads / kWave);
        const int cols = (int)((row_bytes + 16 * kWave - 1) / (16 * kWave));
        auto launch = paced_copy(bytes, row_bytes) ? launch_pipe<kCols, kRowsPerWave, true>
                                                  : launch_pipe<kCols, kRowsPerWave, false>;
        launch(cols, dim3((unsigned)pb), dim3(kThreads), s, src, dst, rows, nout, nrows, row_bytes);
    } else if (!elements) {
        hipLaunchKernelGGL(gather_vec_kernel<kCols>, dim3((unsigned)blocks), dim3(kThreads), 0, s, src, dst, rows,
                           nout, nrows, row_bytes);
    } else if (elem_bytes == 2) {
        hipLaunchKernelGGL(gather_elem_kernel<uint16_t>, dim3((unsigned)blocks), dim3(kThreads), 0, s,
                           static_cast<const uint16_t*>(X), static_cast<uint16_t*>(out), rows, nout,
                           nrows, row_bytes / 2);
    } else {
        hipLaunchKernelGGL(gather_elem_kernel<uint32_t>, dim3((unsigned)blocks), dim3(kThreads), 0, s,
                           static_cast<const uint32_t*>(X), static_cast<uint32_t*>(out), rows, nout,
                           nrows, row_bytes / 4);
    }
    return hipGetLastError();
}

}  // namespace tr
