// Gather of the kept rows: out[r, :] = X[rows[r], :], byte for byte.
// Every lane moves UNR x 16 bytes per step, wherever the rows start (the
// 16-byte accesses take any byte address); a row's last piece is its last 16
// bytes, which overlap the piece before where the row is no multiple of 16
// (both write the same bytes there).  Only rows below 16 bytes go element by
// element.  Rows
// of at most 8 KiB (one step) go two to a wavefront, the second row's loads
// in flight while the first is stored (64 x 576 x 4096 bf16 step: 150.4 ->
// 148.8 us; four rows to a wavefront: 151.6 us); longer rows take one
// wavefront each, all loads of a step issued before its stores.  Loads and
// stores are non-temporal: nothing is reused (non-temporal stores measured
// 8.6 vs 11.2 us for 4096 rows of 8 KiB).
#include "tr_internal.h"

namespace tr {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_any __attribute__((aligned(2)));

__device__ __forceinline__ u32x4 load16(const char* row, int64_t off)
{
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(row + off));
}

__device__ __forceinline__ void store16(char* row, int64_t off, u32x4 v)
{
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4_any*>(row + off));
}

template <int UNR>
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
    const int64_t vec_per_row = (row_bytes + 15) / 16, last = row_bytes - 16;
    for (int64_t j0 = lane; j0 < vec_per_row; j0 += (int64_t)kWave * UNR) {
        u32x4 v[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int64_t j = j0 + (int64_t)kWave * u;
            v[u] = load16(s, j * 16 < last ? j * 16 : last);
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int64_t j = j0 + (int64_t)kWave * u;
            if (j < vec_per_row) store16(d, j * 16 < last ? j * 16 : last, v[u]);
        }
    }
}

// Rows of at most 64 x UNR chunks, RPW consecutive output rows per
// wavefront: the loads of row k + 1 are in flight while row k is stored.
// PACED: they are issued when row k has arrived.  Copies of some tens of MB
// run faster so (4608 rows of 8 KB 14.4 against 15.7 us, 5120 rows 14.5 against
// 15.1), large ones with both rows' loads in flight (29700 rows of 7 KB 79.6
// against 76.0 us).
template <int UNR, int RPW, bool PACED>
__global__ __launch_bounds__(256) void gather_pipe_kernel(const char* __restrict__ X, char* __restrict__ out,
                                                           const int32_t* __restrict__ rows,
                                                           int64_t nout, int64_t nrows, int64_t row_bytes)
{
    const int vec_per_row = (int)((row_bytes + 15) / 16), last = (int)row_bytes - 16;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t r0 = ((int64_t)blockIdx.x * (blockDim.x / kWave) + (threadIdx.x / kWave)) * RPW;
    if (r0 >= nout) return;
    // The source rows first: an index read between the copies would wait for
    // every load before it.
    int64_t src[RPW];
#pragma unroll
    for (int k = 0; k < RPW; ++k) src[k] = rows[r0 + k < nout ? r0 + k : r0];
    u32x4 v[2][UNR];
    auto ok = [&](int k) { return r0 + k < nout && src[k] >= 0 && src[k] < nrows; };   // memory safety against a bad index
    auto load = [&](int k) {
        const char* s = X + (ok(k) ? src[k] : 0) * row_bytes;
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int j = lane + kWave * u;
            v[k & 1][u] = load16(s, j * 16 < last ? j * 16 : last);
        }
    };
    auto store = [&](int k) {
        if (!ok(k)) return;
        char* d = out + (r0 + k) * row_bytes;
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int j = lane + kWave * u;
            if (j < vec_per_row) store16(d, j * 16 < last ? j * 16 : last, v[k & 1][u]);
        }
    };
    load(0);
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
        if (k + 1 < RPW) {
            if constexpr (PACED) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            load(k + 1);
        }
        store(k);
    }
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

}  // namespace

hipError_t launch_gather(const void* X, void* out, const int32_t* rows, int64_t nout, int64_t nrows,
                         int64_t row_bytes, int elem_bytes, hipStream_t s)
{
    if (nout <= 0) return hipSuccess;
    constexpr int kThreads = 256;
    const int64_t blocks = (nout + kThreads / kWave - 1) / (kThreads / kWave);
    constexpr int kUnr = 8, kRowsPerWave = 2;
    const char* src = static_cast<const char*>(X);
    char* dst = static_cast<char*>(out);
    if (row_bytes >= 16 && row_bytes <= 16 * kWave * kUnr) {
        const int64_t waves = (nout + kRowsPerWave - 1) / kRowsPerWave;
        const int64_t pb = (waves + kThreads / kWave - 1) / (kThreads / kWave);
        constexpr int64_t kBurstBytes = 128 << 20;
        if (nout * row_bytes < kBurstBytes)
            hipLaunchKernelGGL((gather_pipe_kernel<kUnr, kRowsPerWave, true>), dim3((unsigned)pb), dim3(kThreads), 0,
                               s, src, dst, rows, nout, nrows, row_bytes);
        else
            hipLaunchKernelGGL((gather_pipe_kernel<kUnr, kRowsPerWave, false>), dim3((unsigned)pb), dim3(kThreads), 0,
                               s, src, dst, rows, nout, nrows, row_bytes);
    } else if (row_bytes >= 16) {
        hipLaunchKernelGGL(gather_vec_kernel<kUnr>, dim3((unsigned)blocks), dim3(kThreads), 0, s, src, dst, rows,
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
