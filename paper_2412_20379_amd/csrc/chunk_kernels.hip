// The copy of a streamed chunk and its weights.
//
// Copy kernel: reads pieces of a chunk (row pointers and lists, column ids, weights if they travel) from pinned host memory
// and writes the device image.  16 blocks keep the link as busy as the DMA engine does (56 GB/s measured for both), and
// it starts in microseconds where a DMA copy takes 20-30; but a kernel that runs beside it waits behind the same memory
// queues (0.07 -> 0.3 ms measured for the weight kernel below), so it is used for what is short: whole
// small chunks, and the row pointers and lists of large ones.
//
// Weights of a streamed chunk rebuilt on the device.  The chunk scheduling of Section 4.2.1 is
// bound by the host link when chunks do not stay resident; for a graph without caller weights the
// stored values follow from the structure alone (the GCN normalisation 1 / sqrt(din(v) dout(u)) of
// Section 4.1.3, or 1), so only the column ids travel and the values are recomputed after the
// copy: half the bytes per chunk.  The arithmetic is the host's, step for step in IEEE double
// (product of the two degrees, square root, reciprocal, one rounding to fp32), so the rebuilt
// values are the stored ones bit for bit.  A block finds the rows of its 4096 entries in a copy of their row pointers in
// LDS (4 M entries of a 306,128-vertex graph: 0.071 -> 0.037 ms).
//
// Column ids travel packed: a vertex id of a graph of 306,128 vertices takes 19 of 32 bits, and the link is what a cold pass
// waits for (15.8 M entries in four chunks, forward and backward: 2.62 -> 1.70 ms).  The unpacking kernel is bound by memory (8 us
// for 4 M ids).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ntp_internal.h"

namespace ntp {

namespace {

constexpr int ENTRIES_PER_BLOCK = 256 * 16;

// largest r in [lo, hi] with rowptr[r] <= e  (rowptr[lo] <= e is given)
__device__ __forceinline__ int64_t row_of(const int64_t* __restrict__ rowptr, int64_t lo, int64_t hi, int64_t e) {
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (rowptr[mid] <= e) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__global__ void __launch_bounds__(256) rebuild_weights_kernel(const int64_t* __restrict__ rowptr, int64_t row_base, int64_t n_rows,
                                                              int64_t e_base, int64_t n_entries, const int32_t* __restrict__ colidx,
                                                              float* __restrict__ val, const int32_t* __restrict__ deg_row,
                                                              const int32_t* __restrict__ deg_col, int mode) {
    __shared__ int64_t span[2];
    __shared__ int32_t start[ENTRIES_PER_BLOCK + 1];       // first entry of each row, relative to this block's first entry
    const int64_t first = (int64_t)blockIdx.x * ENTRIES_PER_BLOCK;
    const int64_t last = std::min<int64_t>(first + ENTRIES_PER_BLOCK, n_entries) - 1;
    if (mode == VAL_ONES) {
        for (int64_t i = first + threadIdx.x; i <= last; i += 256) val[i] = 1.0f;
        return;
    }
    // rows this block's entries lie in (entries are ordered by row); a chunk that holds part of
    // one row has n_rows = 1 and every entry belongs to that row
    if (threadIdx.x < 2) span[threadIdx.x] = row_of(rowptr, 0, n_rows - 1, e_base + (threadIdx.x == 0 ? first : last));
    __syncthreads();
    const int64_t r_lo = span[0], r_hi = span[1];
    const bool in_lds = r_hi - r_lo < ENTRIES_PER_BLOCK;   // always, unless rows without entries lie between
    const int nr = (int)(r_hi - r_lo) + 1;
    if (in_lds) {
        for (int i = threadIdx.x; i < nr; i += 256) start[i] = (int32_t)std::max<int64_t>(rowptr[r_lo + i] - (e_base + first), -1);
        __syncthreads();
    }
    int known = 0;                                          // this thread's entries ascend: so do their rows
    for (int64_t i = first + threadIdx.x; i <= last; i += 256) {
        int64_t r;
        if (in_lds) {
            const int32_t e = (int32_t)(i - first);
            int lo = known, hi = nr - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (start[mid] <= e) lo = mid; else hi = mid - 1;
            }
            known = lo;
            r = r_lo + lo;
        } else {
            r = row_of(rowptr, r_lo, r_hi, e_base + i);
        }
        const double prod = (double)deg_row[row_base + r] * (double)deg_col[colidx[i]];
        const double scale = 1.0 / sqrt(prod);
        val[i] = (float)scale;
    }
}

// four ids a thread
__global__ void __launch_bounds__(256) unpack_ids_kernel(const uint32_t* __restrict__ packed, int bits, int64_t n, int32_t* __restrict__ ids) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= n) return;
    int32_t v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t at = std::min(i + q, n - 1) * bits;
        const uint64_t two = (uint64_t)packed[at >> 5] | (uint64_t)packed[(at >> 5) + 1] << 32;
        v[q] = (int32_t)((uint32_t)(two >> (at & 31)) & ((1u << bits) - 1));
    }
    if (i + 4 <= n) __builtin_memcpy(ids + i, v, 16);
    else
        for (int q = 0; q < 3; ++q)
            if (i + q < n) ids[i + q] = v[q];
}

// up to three pieces; source and destination of a piece have the same address modulo 16
struct StageArgs { const char* src[3]; char* dst[3]; int64_t bytes[3]; };

__global__ void __launch_bounds__(256) stage_kernel(const StageArgs a) {
    const int64_t stride = (int64_t)gridDim.x * 256, t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (int p = 0; p < 3; ++p) {
        const int64_t n = a.bytes[p];
        if (n == 0) continue;
        const int64_t head = std::min<int64_t>(n, (16 - (int64_t)((uintptr_t)a.src[p] % 16)) % 16);
        const int64_t nv = (n - head) / 16, tail = n - head - nv * 16;      // bytes in multiples of 4
        if (t * 4 < head) *reinterpret_cast<int32_t*>(a.dst[p] + t * 4) = *reinterpret_cast<const int32_t*>(a.src[p] + t * 4);
        if (t * 4 < tail) {
            const int64_t o = head + nv * 16 + t * 4;
            *reinterpret_cast<int32_t*>(a.dst[p] + o) = *reinterpret_cast<const int32_t*>(a.src[p] + o);
        }
        const uint4* s = reinterpret_cast<const uint4*>(a.src[p] + head);
        uint4* d = reinterpret_cast<uint4*>(a.dst[p] + head);
        int64_t i = t;
        for (; i + 3 * stride < nv; i += 4 * stride) {
            const uint4 x0 = s[i], x1 = s[i + stride], x2 = s[i + 2 * stride], x3 = s[i + 3 * stride];
            d[i] = x0; d[i + stride] = x1; d[i + 2 * stride] = x2; d[i + 3 * stride] = x3;
        }
        for (; i < nv; i += stride) d[i] = s[i];
    }
}

}  // namespace

int launch_stage_chunk(const void* const src[3], void* const dst[3], const int64_t bytes[3], void* stream) {
    StageArgs a;
    int64_t total = 0;
    for (int p = 0; p < 3; ++p) { a.src[p] = static_cast<const char*>(src[p]); a.dst[p] = static_cast<char*>(dst[p]); a.bytes[p] = bytes[p]; total += bytes[p]; }
    if (total == 0) return NTP_OK;
    const unsigned blocks = (unsigned)std::max<int64_t>(1, std::min<int64_t>(16, (total / 16 + 255) / 256));
    hipLaunchKernelGGL(stage_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, a);
    if (hipGetLastError() != hipSuccess) { set_error("chunk copy kernel launch failed"); return NTP_EHIP; }
    return NTP_OK;
}

int launch_unpack_ids(const uint32_t* packed, int bits, int64_t n, int32_t* ids, void* stream) {
    if (n <= 0) return NTP_OK;
    hipLaunchKernelGGL(unpack_ids_kernel, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, (hipStream_t)stream, packed, bits, n, ids);
    if (hipGetLastError() != hipSuccess) { set_error("column id kernel launch failed"); return NTP_EHIP; }
    return NTP_OK;
}

int launch_rebuild_weights(const int64_t* rowptr, int64_t row_base, int64_t n_rows, int64_t e_base, int64_t n_entries,
                           const int32_t* colidx, float* val, const int32_t* deg_row, const int32_t* deg_col, int mode,
                           void* stream) {
    if (n_entries <= 0) return NTP_OK;
    const int64_t blocks = (n_entries + ENTRIES_PER_BLOCK - 1) / ENTRIES_PER_BLOCK;
    hipLaunchKernelGGL(rebuild_weights_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, rowptr, row_base, n_rows,
                       e_base, n_entries, colidx, val, deg_row, deg_col, mode);
    if (hipGetLastError() != hipSuccess) { set_error("weight rebuild kernel launch failed"); return NTP_EHIP; }
    return NTP_OK;
}

}  // namespace ntp
