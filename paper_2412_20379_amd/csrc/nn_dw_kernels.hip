// Weight gradient of the dense transform: dW[k x m] = A^T dZ, A [n x k], dZ = dH (* 1[H > 0]) [n x m], a contraction
// over the vertices.
//
// Both operands run along their rows in memory and the contraction runs across them, which is what the
// matrix instruction wants when the columns are dealt out differently: a lane that reads VEC consecutive columns of a
// row holds one element of VEC different 32-column blocks, so eight rows read that way are VEC complete operands
// (lane = column, eight contraction indices) with no transposition and no LDS.  A wavefront owns a tile of dW (128 x 64
// where both sides are that wide) and walks its rows 16 at a time: coalesced loads of the next rows are in
// flight while the present ones are cut into bf16 pieces and multiplied; no barrier until the end.  A block of eight
// wavefronts is a few neighbouring tiles x shares of the rows of one range of vertices; the shares are added through
// LDS in a fixed order, the ranges by sum_splits_kernel: deterministic.
//
// Bound: memory for a narrow side (256 x 64 on 169,343 rows: 217 MB in 0.043 ms = 5.0 TB/s), the two pipes of the SIMD
// otherwise (256 x 256: matrix instructions 49 % of the time, other vector instructions 40 %, half of them beside those).
// Against 128 x 128 tiles cut through LDS behind barriers, which this replaces (169,343 rows, fp32, without / with the ReLU
// mask): 256 x 256 0.147 / 0.185 -> 0.139 / 0.161 ms, 128 x 256 0.085 / 0.108 -> 0.074 / 0.097, 256 x 64 0.065 / 0.149 ->
// 0.044 / 0.052, 256 x 40 0.061 / 0.132 -> 0.042 / 0.046; 58,241 rows of 128 x 64 0.037 / 0.070 -> 0.020 / 0.023.
// m <= 32 runs on the fp32 matrix instructions (the rule is in nn_kernels.hip), which bound it as much as memory does:
// 256 x 16 0.042 ms against 0.037 with pieces and 0.044 in the fp32 tiles replaced (masked 0.042 / 0.040 / 0.050).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "nn_util.h"
#include "ntp_internal.h"

namespace ntp {

namespace {

struct DwArgs {
    const void* A;
    const void* Z;         // dH
    const void* mask;      // H (nullable): an element of dH counts only where H > 0
    float* out;            // [n_splits][k x m] partial sums, or dW itself
    int64_t n;
    int k, m;
    int kt, mt;            // wavefront tiles (64 x 32 * TN) of a block: kt * mt in {1, 2, 4, 8}
    int tiles_k, tiles_m;  // block tiles
    int n_splits;
    int64_t rows_per_split;    // multiple of 16
};

// VEC consecutive elements in one load (element alignment is enough)
template <class T, int VEC>
__device__ __forceinline__ void load_vec(const T* p, T (&v)[VEC]) {
    __builtin_memcpy(v, p, sizeof(T) * VEC);
}

// the parts of eight rows of one column block
template <class T, Core C>
__device__ __forceinline__ void cut_rows(const T (&x)[8], uint4 (&piece)[Parts<T, C>::n]) {
    if constexpr (sizeof(T) == 2) {
        unsigned w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (unsigned)x[2 * e] | ((unsigned)x[2 * e + 1] << 16);
        piece[0] = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
        unsigned w[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = __float_as_uint(x[e]);
        cut_row8<T, C>(w, piece);
    }
}

// A wavefront owns 64 columns of A x 32 * TN columns of dZ; the block's eight wavefronts are g.kt x g.mt such tiles x
// row shares.
template <class T, Core C, bool MASK, int VA, int VB, int TA, int TN>
__global__ void __launch_bounds__(512, 2) dw_kernel(const DwArgs g) {
    constexpr bool RING = TA * TN <= 4;        // two steps in flight (else one: the accumulators take the registers)
    constexpr int NP = Parts<T, C>::n;
    extern __shared__ float lds[];             // sums of the row shares
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r = lane & 31, h = lane >> 5;
    const int per_share = g.kt * g.mt, shares = 8 / per_share;
    const int tile = wave % per_share, share = wave / per_share;
    // blocks of one range of vertices have ids that differ by 8: one XCD
    const int minor = g.tiles_k * g.tiles_m, id = (int)blockIdx.x;
    const int split = id / (8 * minor) * 8 + id % 8, t = id / 8 % minor;
    if (split >= g.n_splits) return;
    const int c0 = (t % g.tiles_k * g.kt + tile % g.kt) * (32 * TA), z0 = (t / g.tiles_k * g.mt + tile / g.kt) * (32 * TN);
    const int64_t r0 = split * g.rows_per_split, r1 = min(r0 + g.rows_per_split, g.n);
    const int k = g.k, m = g.m;
    const T* A = static_cast<const T*>(g.A);
    const T* Z = static_cast<const T*>(g.Z);
    const T* M = static_cast<const T*>(g.mask);

    // the first column of each of this lane's vectors; a vector that would cross the edge of the matrix is taken at the edge
    // (its columns are then computed by two lanes, which store the same numbers)
    int ca[TA / VA], cz[TN / VB];
#pragma unroll
    for (int v = 0; v < TA / VA; ++v) ca[v] = min(c0 + 32 * VA * v + VA * r, k - VA);
#pragma unroll
    for (int v = 0; v < TN / VB; ++v) cz[v] = min(z0 + 32 * VB * v + VB * r, m - VB);

    f32x16 acc[TA][TN];
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    struct Raw { T a[8][TA / VA][VA], z[8][TN / VB][VB], mk[MASK ? 8 : 1][TN / VB][VB]; };
    // rows row0 + 2 j + h, j < 8; WHOLE: all of them below r1, else the rows beyond re-read the last one
    auto fetch = [&](Raw& x, int64_t row0, auto whole) {
        constexpr bool WHOLE = decltype(whole)::value;
        const int last = (int)(r1 - 1 - row0);
        const T* zb = Z + row0 * m;
        const T* mb = M + row0 * m;
        const T* ab = A + row0 * k;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            // whole steps: a uniform base per row pair and one lane offset for all of them
            const int row = WHOLE ? h : min(2 * j + h, last);
            const T* zj = WHOLE ? zb + 2 * j * m : zb;
            const T* mj = WHOLE ? mb + 2 * j * m : mb;
            const T* aj = WHOLE ? ab + 2 * j * k : ab;
#pragma unroll
            for (int v = 0; v < TN / VB; ++v) {
                load_vec<T, VB>(zj + (row * m + cz[v]), x.z[j][v]);
                if constexpr (MASK) load_vec<T, VB>(mj + (row * m + cz[v]), x.mk[j][v]);
            }
#pragma unroll
            for (int v = 0; v < TA / VA; ++v) load_vec<T, VA>(aj + (row * k + ca[v]), x.a[j][v]);
        }
    };
    // multiply the rows held in x; left < 16: the rows from the left-th on count as zero.  A non-negative
    // next is the row whose step x is refilled with (a whole one).
    auto use = [&](Raw& x, int left, int64_t next, auto whole) {
        constexpr bool WHOLE = decltype(whole)::value;
        uint4 pb[TN][NP];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            T y[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                y[e] = x.z[e][j / VB][j % VB];
                if constexpr (MASK) y[e] = elem_to_f32(x.mk[e][j / VB][j % VB]) > 0.f ? y[e] : (T)0;
                if constexpr (!WHOLE) y[e] = 2 * e + h < left ? y[e] : (T)0;
            }
            cut_rows<T, C>(y, pb[j]);
        }
        auto cut_a = [&](int i, uint4 (&pa)[NP]) {
            T y[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                y[e] = x.a[e][i / VA][i % VA];
                if constexpr (!WHOLE) y[e] = 2 * e + h < left ? y[e] : (T)0;
            }
            cut_rows<T, C>(y, pa);
        };
        if constexpr (RING) {
            uint4 pa[TA][NP];
#pragma unroll
            for (int i = 0; i < TA; ++i) cut_a(i, pa[i]);
            // pieces leave x free before they are multiplied; floats are multiplied where they were loaded to (602 x 16 on
            // 58,241 rows: 62.2 us, refilled before 64.4)
            if constexpr (WHOLE && C == CORE_BF16) {
                if (next + 16 <= r1) fetch(x, next, whole);
            }
            mfma_parts<C, TA, TN, NP>(pa, pb, acc);
            if constexpr (WHOLE && C == CORE_F32) {
                if (next + 16 <= r1) fetch(x, next, whole);
            }
        } else {
#pragma unroll
            for (int i = 0; i < TA; ++i) {
                uint4 pa[1][NP];
                cut_a(i, pa[0]);
                if constexpr (WHOLE) {
                    if (i == TA - 1 && next + 16 <= r1) fetch(x, next, whole);
                }
                mfma_parts<C, 1, TN, NP>(pa, pb, reinterpret_cast<f32x16 (&)[1][TN]>(acc[i]));
            }
        }
    };
    const std::true_type whole{};
    const std::false_type ragged{};
    const int64_t d = 16 * shares;
    int64_t row = r0 + 16 * share;
    Raw x0;
    if (row + 16 <= r1) fetch(x0, row, whole);
    if constexpr (RING) {
        Raw x1;
        if (row + d + 16 <= r1) fetch(x1, row + d, whole);
        while (row + 16 <= r1) {
            use(x0, 16, row + 2 * d, whole);
            row += d;
            if (row + 16 > r1) break;
            use(x1, 16, row + 2 * d, whole);
            row += d;
        }
    } else {
        for (; row + 16 <= r1; row += d) use(x0, 16, row + d, whole);
    }
    if (row < r1) {            // the last, partial step of the whole range belongs to one share
        fetch(x0, row, ragged);
        use(x0, (int)(r1 - row), 0, ragged);
    }

    // add the row shares: the upper half hands its sums to the lower half until one share is left
    constexpr int TILE = TA * TN * 16 * 64;
    for (int half = shares / 2; half >= 1; half /= 2) {
        if (share >= half && share < 2 * half) {
            float* dst = lds + ((share - half) * per_share + tile) * TILE + lane;
#pragma unroll
            for (int i = 0; i < TA; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) dst[((i * TN + j) * 16 + e) * 64] = acc[i][j][e];
        }
        __syncthreads();
        if (share < half) {
            const float* src = lds + (share * per_share + tile) * TILE + lane;
#pragma unroll
            for (int i = 0; i < TA; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[i][j][e] += src[((i * TN + j) * 16 + e) * 64];
        }
        __syncthreads();
    }
    if (share == 0) {
        // element e of a 32x32 block: row 8*(e/4) + 4*(lane/32) + e%4 of the A columns, column lane%32 of dZ's
        float* out = g.out + (int64_t)split * k * m;
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = cz[j / VB] + j % VB;
                const bool in = z0 + 32 * VB * (j / VB) + VB * r < m;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int first = c0 + 32 * VA * (i / VA) + VA * (8 * (e / 4) + 4 * h + e % 4);
                    if (in && first < k) out[(int64_t)(min(first, k - VA) + i % VA) * m + col] = acc[i][j][e];
                }
            }
    }
}

template <class T, Core C, bool MASK, int VA, int VB, int TA, int TN>
void launch_dw(const DwArgs& g, hipStream_t st) {
    constexpr int lds = 4 * TA * TN * 16 * 64 * 4;          // the upper half of the wavefronts' sums
    auto kernel = dw_kernel<T, C, MASK, VA, VB, TA, TN>;
    static bool allowed[64] = {};
    int dev = 0;
    (void)hipGetDevice(&dev);
    if (dev >= 0 && dev < 64 && !allowed[dev])
        allowed[dev] = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds) == hipSuccess;
    const int64_t blocks = (int64_t)(g.n_splits + 7) / 8 * 8 * g.tiles_k * g.tiles_m;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(512), lds, st, g);
}

int pow2_up(int64_t x, int most) {
    int p = 1;
    while (p < most && p < x) p <<= 1;
    return p;
}

// The shape of a wavefront tile and how the work is cut.
//   k < 4 (no whole vector of four columns of A): 32 x 32 read element by element, up to eight column tiles side by side
//     (2 x 64 on 306,129 rows 0.025 ms against 0.111 in tiles through LDS, 3 x 256 0.077 against 0.186);
//   m <= 32: 128 x 32, on the fp32 instructions 32 x 32 for k <= 32 (padding is dear there: 16 x 16 on 300,000 rows 17.4
//     against 39.1 us);
//   k <= 64 < m: 64 x 64 (a 128-column tile would be mostly padding);
//   else 128 x 64, whose operands are cut into pieces for 48 matrix instructions instead of 24 a step: 256 x 256 on 169,343
//     rows 0.134 against 0.164 ms.
// m <= 32 and more than three row tiles of A take four of them side by side: whole rows of A from few blocks (us with one /
// four, 602 x 16 on 16,000 rows 27.3 / 22.5, 50,000 54.7 / 46.9, 200,000 195 / 162; 1433 x 16 on 30,000 75.2 / 70.5; 256 x 16
// on 120,000 33.6 / 35.5, so not there; 602 x 16 on 8,000 13.9 / 16.4: the few rows of a block are better shared out).
// Blocks: about one per compute unit; two column tiles side by side where there are two (they share the rows of A through the
// L1), the other wavefronts share out the rows.
enum { DW_NARROW, DW_SHORT, DW_WIDE, DW_TINY };
int dw_shape(int64_t k, int64_t m, bool fp32_core) {
    if (k < 4) return DW_TINY;
    if (m > 32) return k <= 64 ? DW_SHORT : DW_WIDE;
    return fp32_core && k <= 32 ? DW_TINY : DW_NARROW;
}

DwArgs dw_plan(int64_t n, int64_t k, int64_t m, bool fp32_core) {
    DwArgs g{};
    g.n = n; g.k = (int)k; g.m = (int)m;
    const int shape = dw_shape(k, m, fp32_core);
    const int ta = shape == DW_TINY ? 1 : shape == DW_SHORT ? 2 : 4, tn = shape == DW_TINY || shape == DW_NARROW ? 1 : 2;
    g.kt = shape == DW_NARROW && k > 384 && n > 10000 ? 4 : 1;
    g.mt = shape == DW_NARROW ? 1 : pow2_up((m + 32 * tn - 1) / (32 * tn), shape == DW_TINY ? 8 : shape == DW_SHORT ? 4 : 2);
    g.tiles_k = (int)((k + 32 * ta * g.kt - 1) / (32 * ta * g.kt));
    g.tiles_m = (int)((m + 32 * tn * g.mt - 1) / (32 * tn * g.mt));
    const int64_t shares = 8 / (g.kt * g.mt), tiles = (int64_t)g.tiles_k * g.tiles_m;
    int64_t s = std::max<int64_t>(1, compute_units() / tiles);
    s = std::min(s, (n + 32 * shares - 1) / (32 * shares));        // at least two steps a wavefront
    if (k < 4) s = std::min(s, std::max<int64_t>(1, n / 256));     // many column tiles: no more partial sums than rows pay for
    g.rows_per_split = ((n + s - 1) / s + 15) / 16 * 16;
    g.n_splits = (int)((n + g.rows_per_split - 1) / g.rows_per_split);
    return g;
}

template <class T, Core C>
void launch_dw_any(const DwArgs& g, hipStream_t st) {
    switch (dw_shape(g.k, g.m, C == CORE_F32)) {
        case DW_TINY:
            if constexpr (sizeof(T) == 2 || C == CORE_F32) g.mask ? launch_dw<T, C, true, 1, 1, 1, 1>(g, st) : launch_dw<T, C, false, 1, 1, 1, 1>(g, st);
            break;
        case DW_NARROW: g.mask ? launch_dw<T, C, true, 4, 1, 4, 1>(g, st) : launch_dw<T, C, false, 4, 1, 4, 1>(g, st); break;
        case DW_SHORT: g.mask ? launch_dw<T, C, true, 2, 2, 2, 2>(g, st) : launch_dw<T, C, false, 2, 2, 2, 2>(g, st); break;
        default: g.mask ? launch_dw<T, C, true, 4, 2, 4, 2>(g, st) : launch_dw<T, C, false, 4, 2, 4, 2>(g, st); break;
    }
}

}  // namespace

// fp32 operands with so few columns have a kernel on the fp32 instructions only (they are bound by reading dZ)
bool nn_dw_fp32_only(int64_t k) { return k < 4; }

int nn_dw_splits(int64_t n, int64_t k, int64_t m, bool fp32_core) { return dw_plan(n, k, m, fp32_core).n_splits; }

// partial sums of every range of vertices to out [splits][k x m]; fp32_core: fp32 operands on the fp32 matrix instructions
int launch_nn_dw(const void* A, const void* dH, const void* mask, float* out, int64_t n, int64_t k, int64_t m, int dtype,
                 bool fp32_core, void* stream) {
    DwArgs g = dw_plan(n, k, m, fp32_core);
    g.A = A; g.Z = dH; g.mask = mask; g.out = out;
    const hipStream_t st = (hipStream_t)stream;
    if (dtype == NTP_BF16) launch_dw_any<unsigned short, CORE_BF16>(g, st);
    else if (fp32_core) launch_dw_any<float, CORE_F32>(g, st);
    else launch_dw_any<float, CORE_BF16>(g, st);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("transform kernel launch failed: %s", hipGetErrorString(e)); return NTP_EHIP; }
    return NTP_OK;
}

}  // namespace ntp
