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
// Column ids travel packed, as the link is what a cold pass waits for: 15.8 M entries of 306,128 vertices in four chunks, forward and
// backward, 2.62 ms as they are, 1.70 in the 19 bits of a vertex id, 1.25 as Elias-Fano parts of the ascending rows (12.7 bits: a row of d
// neighbours among n vertices needs log2(n / d) + 1.5 bits an id at least, and many entries are in long rows).  Blocks of 256 entries, by entries and not by rows: each its
// own number of low bits, so that hubs and short rows both come out near what they need, and a wavefront a block (of 128, 512 and 1,024 entries 12.8, 12.9 and
// 13.2 bits).  The unpacking kernel takes 15.5 us for 4 M ids, 8 in plain bits; its chain of loads bounds it, and it runs beside the next copy.
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

// A wavefront a block of PACK_BLOCK entries, four a lane.  The ones of the bit string are found 16 places a lane, behind a scan over the words'
// counts, and leave their entry's high part in LDS; nothing is waited for but the block's own words.
__global__ void __launch_bounds__(256) unpack_ids_kernel(const uint32_t* __restrict__ packed, int bits, int64_t n_cols, double per_col, int64_t n,
                                                         int32_t* __restrict__ ids) {
    static_assert(PACK_BLOCK == 256, "four entries a lane");
    __shared__ __align__(8) uint16_t high_lds[4][PACK_BLOCK];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t block = (int64_t)blockIdx.x * 4 + wave;
    if (block * PACK_BLOCK >= n) return;
    const int len = (int)std::min<int64_t>(PACK_BLOCK, n - block * PACK_BLOCK);
    const uint32_t begin = packed[block], end = packed[block + 1];
    const uint32_t* w = packed + begin;
    const uint32_t first = w[0];
    const int l = (int)w[1];
    w += 2;
    const bool plain = l == PACK_PLAIN;
    const int lb = plain ? bits : l;
    const int n_low = (len * lb + 31) / 32, n_high = (int)(end - begin) - 2 - n_low;      // n_high <= (len + 2 len + 1 + 31) / 32 < 32
    const uint32_t* low = w + n_high;
    const int i0 = lane * 4;
    uint32_t v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int at = std::min(i0 + q, len - 1) * lb;
        const uint64_t two = (uint64_t)low[at >> 5] | (uint64_t)low[(at >> 5) + 1] << 32;
        v[q] = (uint32_t)(two >> (at & 31)) & ((1u << lb) - 1);
    }
    if (!plain) {
        uint16_t* const high = high_lds[wave];
        const uint32_t word = lane < n_high ? w[lane] : 0u;
        int before = __popc(word);                        // ones up to this word's end, then up to its start
        for (int d = 1; d < 32; d *= 2) {
            const int x = __shfl_up(before, d);
            before += lane >= d ? x : 0;
        }
        before -= __popc(word);
        const uint32_t mine = __shfl(word, lane / 2);
        int rank = __shfl(before, lane / 2);
        uint32_t ones = mine;
        if (lane & 1) { rank += __popc(mine & 0xffffu); ones &= 0xffff0000u; }
        else ones &= 0xffffu;
        while (ones) {
            const int at = (lane / 2) * 32 + __ffs(ones) - 1;
            if (rank < PACK_BLOCK) high[rank] = (uint16_t)(at - rank);
            ++rank;
            ones &= ones - 1;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");       // the lanes read what other lanes wrote (in order in the hardware)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t z = ((int64_t)high[i0 + q] << l) + v[q] + first;       // less than (PACK_BLOCK + 1) * n_cols
            int64_t id = z - (int64_t)((double)z * per_col) * n_cols;            // the quotient to within one
            id += id < 0 ? n_cols : 0;
            id -= id >= n_cols ? n_cols : 0;
            v[q] = (uint32_t)id;
        }
    }
    int32_t* const out = ids + block * PACK_BLOCK + i0;
    if (i0 + 4 <= len) __builtin_memcpy(out, v, 16);
    else
#pragma unroll
        for (int q = 0; q < 3; ++q)
            if (i0 + q < len) out[q] = (int32_t)v[q];
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

int launch_unpack_ids(const uint32_t* packed, int bits, int64_t n_cols, int64_t n, int32_t* ids, void* stream) {
    if (n <= 0) return NTP_OK;
    const int64_t blocks = (n + PACK_BLOCK - 1) / PACK_BLOCK;
    hipLaunchKernelGGL(unpack_ids_kernel, dim3((unsigned)((blocks + 3) / 4)), dim3(256), 0, (hipStream_t)stream, packed, bits, n_cols,
                       1.0 / (double)std::max<int64_t>(1, n_cols), n, ids);
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
