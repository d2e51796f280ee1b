// Construction of the topology on the device, for graphs that stay there: the forms of build_host_graph (graph_build.cpp), bit for bit, from an edge
// list without weights.  Without weights the entries of a row that are equal cannot be told apart, so the processing order of the host
// build (input order, reversed copies, self loops) is any stable order: the entries are sorted by (row, neighbour) as numbers.
//
// Keys row * 2^b + neighbour (b bits hold a vertex id), one per input edge, reversed copy and self loop; least significant digit first in
// passes of up to 9 bits: digit counts of every tile of 4,096 keys, their prefix sums, and a stable scatter that orders a tile in LDS so
// that runs of equal digits are written side by side.  Dropping repeated keys, row pointers and column ids follow in one sweep.  The form by source is
// the same entries, already in order of their destination, after the passes over the source's bits alone.
//
// Bound: what surrounds it.  1.2 M edges symmetrised with self loops (2.5 M keys of 36 bits, four passes), 1.7 ms in all: the edges come in in 0.34, keys,
// sorting and arrays take 0.19, row pointers go back in 0.13, allocation and release of 45 MB take 0.5, the plan of the rows on the host 0.5; the
// threads' build took 3.9 and the upload of its arrays 0.8.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ntp_internal.h"

namespace ntp {

namespace {

constexpr int RADIX_BITS = BUILD_RADIX_BITS, RADIX = 1 << RADIX_BITS;
constexpr int TILE = BUILD_TILE, ITEMS = TILE / 256;
typedef unsigned long long u64;

__global__ void __launch_bounds__(256) make_keys_kernel(const int32_t* __restrict__ src, const int32_t* __restrict__ dst, int64_t edges, int64_t n, int bits,
                                                        bool symmetrise, bool loops, u64* __restrict__ keys, u64* __restrict__ bad) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < edges) {
        const int32_t s = src[i], d = dst[i];
        const bool ok = s >= 0 && s < n && d >= 0 && d < n;
        if (!ok) atomicMin(bad, (u64)i);
        keys[i] = ok ? (u64)d << bits | (u64)s : 0;
        if (symmetrise) keys[edges + i] = ok ? (u64)s << bits | (u64)d : 0;
    } else if (loops && i < edges + n) {
        const u64 v = (u64)(i - edges);
        keys[(symmetrise ? edges : 0) + i] = v << bits | v;
    }
}

__global__ void __launch_bounds__(256) digit_counts_kernel(const u64* __restrict__ keys, int64_t count, int shift, int digits, int tiles, int32_t* __restrict__ counts) {
    __shared__ int32_t hist[RADIX];
    for (int d = threadIdx.x; d < digits; d += 256) hist[d] = 0;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * TILE, end = min(first + TILE, count);
    for (int64_t i = first + threadIdx.x; i < end; i += 256) atomicAdd(&hist[(keys[i] >> shift) & (digits - 1)], 1);
    __syncthreads();
    for (int d = threadIdx.x; d < digits; d += 256) counts[(int64_t)d * tiles + blockIdx.x] = hist[d];
}

// exclusive prefix sum over a block's 256 threads; returns the total
__device__ __forceinline__ int block_prefix(int v, int* before, int* lds) {          // lds: 4 ints
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == 63) lds[wave] = x;
    __syncthreads();
    int base = 0, total = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w < wave) base += lds[w];
        total += lds[w];
    }
    __syncthreads();
    *before = base + x - v;
    return total;
}

// row d of counts becomes its exclusive prefix sums; totals[d] its sum
__global__ void __launch_bounds__(256) scan_counts_kernel(int32_t* __restrict__ counts, int tiles, int32_t* __restrict__ totals) {
    __shared__ int lds[4];
    int32_t* row = counts + (int64_t)blockIdx.x * tiles;
    int sum = 0;
    for (int t0 = 0; t0 < tiles; t0 += 256) {
        const int t = t0 + (int)threadIdx.x, v = t < tiles ? row[t] : 0;
        int before;
        const int all = block_prefix(v, &before, lds);
        if (t < tiles) row[t] = sum + before;
        sum += all;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = sum;
}

__global__ void __launch_bounds__(256) scatter_kernel(const u64* __restrict__ keys, int64_t count, int shift, int digits, int tiles,
                                                      const int32_t* __restrict__ counts, const int32_t* __restrict__ totals, u64* __restrict__ out) {
    __shared__ u64 sorted[TILE];
    __shared__ int32_t seen[4][RADIX];                 // per wavefront: keys of a digit so far, then the place of its first one in the tile
    __shared__ int32_t to[RADIX];                      // where a digit's keys of this tile go, less their place in the tile
    __shared__ int lds[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int d = tid; d < 4 * RADIX; d += 256) (&seen[0][0])[d] = 0;
    __syncthreads();
    // a wavefront ranks its quarter of the tile in order, 64 keys at a time: those of the same digit by lane
    const int64_t first = (int64_t)blockIdx.x * TILE + wave * (64 * ITEMS);
    u64 key[ITEMS];
    int rank[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t at = first + i * 64 + lane;
        key[i] = at < count ? keys[at] : 0;
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool in = first + i * 64 + lane < count;
        const int d = (int)(key[i] >> shift) & (digits - 1);
        u64 same = __ballot(in);
#pragma unroll
        for (int b = 0; b < RADIX_BITS; ++b) {
            const u64 set = __ballot((d >> b) & 1);
            same &= (d >> b) & 1 ? set : ~set;
        }
        const int below = __popcll(same & ((1ull << lane) - 1));
        int before = 0;
        if (in) before = seen[wave][d];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (in && below == 0) seen[wave][d] = before + __popcll(same);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        rank[i] = before + below;
    }
    __syncthreads();
    // two digits a thread: places in the tile, places in the output
    int of[2], before;
#pragma unroll
    for (int q = 0; q < 2; ++q) of[q] = seen[0][2 * tid + q] + seen[1][2 * tid + q] + seen[2][2 * tid + q] + seen[3][2 * tid + q];
    block_prefix(of[0] + of[1], &before, lds);
    int global[2] = {0, 0}, global_before;
#pragma unroll
    for (int q = 0; q < 2; ++q) global[q] = 2 * tid + q < digits ? totals[2 * tid + q] : 0;
    block_prefix(global[0] + global[1], &global_before, lds);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int d = 2 * tid + q;
        int place = before;
        if (d < digits) to[d] = global_before + counts[(int64_t)d * tiles + blockIdx.x] - place;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int c = seen[w][d];
            seen[w][d] = place;
            place += c;
        }
        before = place;
        global_before += global[q];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (first + i * 64 + lane < count) sorted[seen[wave][(int)(key[i] >> shift) & (digits - 1)] + rank[i]] = key[i];
    __syncthreads();
    const int mine = (int)min((int64_t)TILE, count - (int64_t)blockIdx.x * TILE);
    for (int j = tid; j < mine; j += 256) {
        const u64 k = sorted[j];
        out[to[(int)(k >> shift) & (digits - 1)] + j] = k;
    }
}

// Which of the sorted keys are entries: with `dedup` the first of equal ones, and self loops only where they were added (`loops`)
struct Keep {
    bool dedup, loops;
    int bits;
    __device__ __forceinline__ bool operator()(const u64* __restrict__ keys, int64_t i) const {
        if (!dedup) return true;
        const u64 k = keys[i];
        if (i > 0 && keys[i - 1] == k) return false;
        return loops || (k >> bits) != (k & ((1ull << bits) - 1));
    }
};

__global__ void __launch_bounds__(256) count_entries_kernel(const u64* __restrict__ keys, int64_t count, Keep keep, int32_t* __restrict__ kept) {
    __shared__ int lds[4];
    const int64_t first = (int64_t)blockIdx.x * TILE;
    int mine = 0, before;
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t at = first + i * 256 + threadIdx.x;
        if (at < count && keep(keys, at)) ++mine;
    }
    const int all = block_prefix(mine, &before, lds);
    if (threadIdx.x == 0) kept[blockIdx.x] = all;
}

// Column ids and row pointers; the key of the transposed entry, where wanted.  kept: exclusive prefix sums over the tiles, total: their sum.
__global__ void __launch_bounds__(256) write_entries_kernel(const u64* __restrict__ keys, int64_t count, int64_t n, Keep keep, const int32_t* __restrict__ kept,
                                                            const int32_t* __restrict__ total, int64_t* __restrict__ rowptr, int32_t* __restrict__ colidx,
                                                            u64* __restrict__ transposed) {
    __shared__ int lds[4];
    const u64 mask = (1ull << keep.bits) - 1;
    const int64_t first = (int64_t)blockIdx.x * TILE;
    int64_t base = kept[blockIdx.x];
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t at = first + i * 256 + threadIdx.x;
        const bool in = at < count, is = in && keep(keys, at);
        int before;
        const int all = block_prefix(is ? 1 : 0, &before, lds);
        if (in) {
            const u64 k = keys[at];
            const int64_t p = base + before, row = (int64_t)(k >> keep.bits);
            if (is) {
                colidx[p] = (int32_t)(k & mask);
                if (transposed) transposed[p] = (k & mask) << keep.bits | (u64)row;
            }
            if (at == 0 || (int64_t)(keys[at - 1] >> keep.bits) != row) rowptr[row] = p;          // p entries come before the row's first key
            if (at == count - 1) rowptr[n] = *total;
        }
        base += all;
    }
}

// Rows without a key (where self loops are added there are none): -1 beforehand, afterwards the row pointer of the next row that has one, found in the
// sorted keys.  One thread a row: a thread that writes all rows between two keys writes up to n of them one after the other (100,000 edges among the
// first 100 of 5 M ids: the build 312 ms, so 54; the threads' build 82).
__global__ void __launch_bounds__(256) mark_rows_kernel(int64_t* __restrict__ rowptr, int64_t n) {
    for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < n; r += (int64_t)gridDim.x * 256) rowptr[r] = -1;
}

__global__ void __launch_bounds__(256) empty_rows_kernel(const u64* __restrict__ keys, int64_t count, int64_t n, int bits, const int32_t* __restrict__ total, int64_t* rowptr) {
    for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < n; r += (int64_t)gridDim.x * 256) {
        if (rowptr[r] >= 0) continue;
        int64_t lo = 0, hi = count;                // the first key of a row beyond r
        while (lo < hi) {
            const int64_t mid = (lo + hi) / 2;
            if ((int64_t)(keys[mid] >> bits) < r) lo = mid + 1;
            else hi = mid;
        }
        rowptr[r] = lo < count ? rowptr[keys[lo] >> bits] : *total;
    }
}

// Row lengths and the longest.  Bound by the additions to one address, so there is one a block and few blocks: 169,343 rows 33 -> 6 us with one a wavefront
// of 64 rows before.
__global__ void __launch_bounds__(256) degrees_kernel(const int64_t* __restrict__ rowptr, int64_t n, int32_t* __restrict__ deg, int32_t* __restrict__ most) {
    __shared__ int32_t longest[4];
    int m = 0;
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < n; v += (int64_t)gridDim.x * 256) {
        const int d = (int)(rowptr[v + 1] - rowptr[v]);
        deg[v] = d;
        m = max(m, d);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = max(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) longest[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(most, max(max(longest[0], longest[1]), max(longest[2], longest[3])));
}

// How often a column occurs.  Bound by the additions to one address where a source has many edges (12 ns each), so a block counts in LDS, each column in
// the place that the first one to come took, and adds a place's count once; columns that find their place taken are added at once.  ms a build of
// 4 M entries without a second form, additions to memory alone / so: of one source 48.3 / 2.6, a third of one source 16.4 / 2.8, of 100,000 alike 2.9 / 2.8 (the host's threads: 6.7).
constexpr int COUNT_BITS = 11, COUNT_ENTRIES = 8192;
__global__ void __launch_bounds__(256) column_counts_kernel(const int32_t* __restrict__ colidx, int64_t nnz, int32_t* __restrict__ counts) {
    __shared__ int32_t column[1 << COUNT_BITS], seen[1 << COUNT_BITS];
    for (int p = threadIdx.x; p < 1 << COUNT_BITS; p += 256) { column[p] = -1; seen[p] = 0; }
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nnz; i += (int64_t)gridDim.x * 256) {
        const int32_t c = colidx[i];
        const unsigned p = (unsigned)c * 2654435761u >> (32 - COUNT_BITS);
        int32_t there = __hip_atomic_load(&column[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (there == -1) there = atomicCAS(&column[p], -1, c);
        if (there == -1 || there == c) atomicAdd(&seen[p], 1);
        else atomicAdd(&counts[c], 1);
    }
    __syncthreads();
    for (int p = threadIdx.x; p < 1 << COUNT_BITS; p += 256)
        if (seen[p]) atomicAdd(&counts[column[p]], seen[p]);
}

__global__ void __launch_bounds__(256) zero_kernel(int32_t* __restrict__ p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0;
}

__global__ void __launch_bounds__(256) compare_kernel(const int32_t* __restrict__ a, const int32_t* __restrict__ b, int64_t n, u64* __restrict__ differ) {
    bool d = false;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) d = d || a[i] != b[i];
    if (__ballot(d) && (threadIdx.x & 63) == 0) atomicMin(differ, 0ull);
}

unsigned blocks_for(int64_t n, int64_t per_block) { return (unsigned)std::max<int64_t>(1, (n + per_block - 1) / per_block); }
unsigned few_blocks(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096)); }

#define HIP_TRY(expr)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess) {                                                              \
            set_error("%s failed: %s", #expr, hipGetErrorString(e_));                        \
            return NTP_EHIP;                                                                 \
        }                                                                                    \
    } while (0)

// `count` keys in `*a` sorted by the bits [lo, hi); `*b`: as much memory.  The sorted ones are in `*a` afterwards.
void sort_keys(u64** a, u64** b, int64_t count, int lo, int hi, int32_t* counts, int32_t* totals) {
    const int tiles = (int)((count + TILE - 1) / TILE), passes = (hi - lo + RADIX_BITS - 1) / RADIX_BITS, width = (hi - lo + passes - 1) / passes;
    for (int shift = lo; shift < hi; shift += width) {
        const int digits = 1 << std::min(width, hi - shift);
        hipLaunchKernelGGL(digit_counts_kernel, dim3((unsigned)tiles), dim3(256), 0, nullptr, *a, count, shift, digits, tiles, counts);
        hipLaunchKernelGGL(scan_counts_kernel, dim3((unsigned)digits), dim3(256), 0, nullptr, counts, tiles, totals);
        hipLaunchKernelGGL(scatter_kernel, dim3((unsigned)tiles), dim3(256), 0, nullptr, *a, count, shift, digits, tiles, counts, totals, *b);
        std::swap(*a, *b);
    }
}

// Row pointers, column ids and, where wanted, the transposed keys of the entries among `count` sorted keys; `kept`: a count a tile
void write_form(const u64* keys, int64_t count, int64_t n, Keep keep, int32_t* kept, int32_t* total, int64_t* rowptr, int32_t* colidx, u64* transposed) {
    const unsigned tiles = (unsigned)((count + TILE - 1) / TILE);
    hipLaunchKernelGGL(count_entries_kernel, dim3(tiles), dim3(256), 0, nullptr, keys, count, keep, kept);
    hipLaunchKernelGGL(scan_counts_kernel, dim3(1), dim3(256), 0, nullptr, kept, (int)tiles, total);
    if (!keep.loops) hipLaunchKernelGGL(mark_rows_kernel, dim3(few_blocks(n)), dim3(256), 0, nullptr, rowptr, n);
    hipLaunchKernelGGL(write_entries_kernel, dim3(tiles), dim3(256), 0, nullptr, keys, count, n, keep, kept, total, rowptr, colidx, transposed);
    if (!keep.loops) hipLaunchKernelGGL(empty_rows_kernel, dim3(few_blocks(n)), dim3(256), 0, nullptr, keys, count, n, keep.bits, total, rowptr);
}

}  // namespace

// Where graphs are built on the device rather than by the host's threads (16 of them): build, export of the arrays and release in us, host / device.
// 2,000 vertices 10,000 edges 253 / 396, 5,000 of 30,000 527 / 319, 10,000 of 100,000 1396 / 488, 50,000 of 300,000 2687 / 1795 (directed 3518 /
// 1555), 169,343 of 1.2 M 7500 / 3390, 1 M of 1 M 15845 / 8252 (directed 32155 / 12792), 200,000 of 4 M 18921 / 10853 (23500 / 9480).  Few edges among many
// vertices, without the export: 200,000 of 24,576 2360 / 1530, 1 M of 24,576 6440 / 3620 (without self loops and with a form by source 8770 / 6580), 20 M of 24,576 196,000 /
// 108,000 (317,000 / 209,000), and 5 M of 100,000 among the first 100 ids 82,000 / 54,000.
// Keys are counted in 32 bits.
bool device_build_takes(int64_t n, int64_t n_edges, uint32_t flags) {
    const int64_t raw = n_edges * (flags & NTP_SYMMETRISE ? 2 : 1) + (flags & NTP_ADD_SELF_LOOPS ? n : 0);
    return n_edges >= 24576 && raw < (1ll << 30) && n >= 2 && n <= (1 << 30);
}

void DeviceForms::release() {
    if (arena) (void)hipFree(arena);
    arena = nullptr;
}

int build_device_forms(int64_t n, int64_t n_edges, const int32_t* src, const int32_t* dst, uint32_t flags, BuiltGraph* g, DeviceForms* out) {
    const bool symmetrise = flags & NTP_SYMMETRISE, dedup = flags & NTP_DEDUP, loops = flags & NTP_ADD_SELF_LOOPS;
    const bool want_csc = !symmetrise && !(flags & NTP_SCATTER_BWD);
    const int bits = bits_of_ids(n);
    const BuildArena arena = plan_build_arena(n, n_edges, flags);
    const int64_t raw = arena.raw;
    const int64_t tiles = (raw + TILE - 1) / TILE;

    // (an arena's size is left for the graph, which takes less in one chunk)
    size_t free_bytes = 0, all_bytes = 0;
    void* p = nullptr;
    if (hipMemGetInfo(&free_bytes, &all_bytes) != hipSuccess || free_bytes / 2 < arena.bytes || hipMalloc(&p, arena.bytes) != hipSuccess) { (void)hipGetLastError(); return DEVICE_BUILD_NO_MEMORY; }
    char* const base = out->arena = static_cast<char*>(p);
    u64 *a = reinterpret_cast<u64*>(base + arena.keys[0]), *b = reinterpret_cast<u64*>(base + arena.keys[1]);
    int32_t *d_src = reinterpret_cast<int32_t*>(b), *d_dst = d_src + n_edges;
    int32_t *counts = reinterpret_cast<int32_t*>(base + arena.counts), *totals = reinterpret_cast<int32_t*>(base + arena.totals), *kept = reinterpret_cast<int32_t*>(base + arena.kept);
    struct Result { u64 bad, differ; int32_t total, most[2], pad; };
    Result* const d_result = reinterpret_cast<Result*>(base + arena.result);
    static_assert(sizeof(Result) <= BUILD_RESULT_BYTES, "the arena holds it");
    int64_t* rowptr[2] = {nullptr, nullptr};
    for (int k = 0; k < arena.row_pointers; ++k) rowptr[k] = reinterpret_cast<int64_t*>(base + arena.rowptr[k]);
    for (int k = 0; k < arena.degrees; ++k) out->degree[k] = reinterpret_cast<int32_t*>(base + arena.degree[k]);
    Result result{~0ull, ~0ull, 0, {0, 0}, 0};
    HIP_TRY(hipMemcpy(d_result, &result, sizeof result, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(d_src, src, (size_t)n_edges * 4, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(d_dst, dst, (size_t)n_edges * 4, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(make_keys_kernel, dim3(blocks_for(n_edges + (loops ? n : 0), 256)), dim3(256), 0, nullptr, d_src, d_dst, n_edges, n, bits, symmetrise, loops, a, &d_result->bad);
    sort_keys(&a, &b, raw, 0, 2 * bits, counts, totals);
    const Keep keep{dedup, loops, bits};
    out->colidx[0] = want_csc ? reinterpret_cast<int32_t*>(base + arena.colidx) : reinterpret_cast<int32_t*>(b);
    write_form(a, raw, n, keep, kept, &d_result->total, rowptr[0], out->colidx[0], want_csc ? b : nullptr);
    hipLaunchKernelGGL(degrees_kernel, dim3(std::min(blocks_for(n, 256), 256u)), dim3(256), 0, nullptr, rowptr[0], n, out->degree[0], &d_result->most[0]);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpy(&result, d_result, sizeof result, hipMemcpyDeviceToHost));
    if (result.bad != ~0ull) {
        set_error("edge %lld has a vertex id outside [0, %lld)", (long long)result.bad, (long long)n);
        return NTP_EINVAL;
    }
    const int64_t nnz = result.total;
    auto host_form = [&](HostSparse& m, int k) {
        m.n = n;
        m.nnz = nnz;
        m.rowptr.resize((size_t)n + 1);
        m.max_degree = result.most[k];
        HIP_TRY(hipMemcpy(m.rowptr.data(), rowptr[k], (size_t)(n + 1) * 8, hipMemcpyDeviceToHost));
        return NTP_OK;
    };
    int rc = host_form(g->csr, 0);
    if (rc != NTP_OK) return rc;
    bool same = symmetrise;
    if (want_csc) {
        if (nnz > 0) {
            sort_keys(&b, &a, nnz, bits, 2 * bits, counts, totals);
            out->colidx[1] = reinterpret_cast<int32_t*>(a);
            write_form(b, nnz, n, Keep{false, loops, bits}, kept, &d_result->total, rowptr[1], out->colidx[1], nullptr);
        } else {
            hipLaunchKernelGGL(zero_kernel, dim3(few_blocks(2 * n)), dim3(256), 0, nullptr, reinterpret_cast<int32_t*>(rowptr[1]), 2 * (n + 1));
        }
        hipLaunchKernelGGL(degrees_kernel, dim3(std::min(blocks_for(n, 256), 256u)), dim3(256), 0, nullptr, rowptr[1], n, out->degree[1], &d_result->most[1]);
        // the same structure has the same weights
        hipLaunchKernelGGL(compare_kernel, dim3(few_blocks(nnz)), dim3(256), 0, nullptr, out->colidx[0], out->colidx[1], nnz, &d_result->differ);
        hipLaunchKernelGGL(compare_kernel, dim3(few_blocks(n)), dim3(256), 0, nullptr, out->degree[0], out->degree[1], n, &d_result->differ);
        HIP_TRY(hipGetLastError());
        HIP_TRY(hipMemcpy(&result, d_result, sizeof result, hipMemcpyDeviceToHost));
        same = result.differ == ~0ull;
        if (!same && (rc = host_form(g->csc, 1)) != NTP_OK) return rc;
    } else if (!symmetrise) {          // only the row lengths of the form by source
        hipLaunchKernelGGL(zero_kernel, dim3(few_blocks(n)), dim3(256), 0, nullptr, out->degree[1], n);
        hipLaunchKernelGGL(column_counts_kernel, dim3(std::min(blocks_for(nnz, COUNT_ENTRIES), 2048u)), dim3(256), 0, nullptr, out->colidx[0], nnz, out->degree[1]);
        HIP_TRY(hipGetLastError());
    }
    if (same) out->degree[1] = out->degree[0];
    g->n = n;
    g->symmetric = same;
    g->has_csc = same || want_csc;
    g->val_mode = flags & NTP_NORM_GCN_SYM ? VAL_GCN : VAL_ONES;
    return NTP_OK;
}

}  // namespace ntp
