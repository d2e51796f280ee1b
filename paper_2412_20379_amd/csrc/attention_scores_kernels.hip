// The vertex-associated half of the GAT attention of Section 2.1: the mapping a^T [W h_u || W h_v]
// splits into two per-vertex scalars, p[v] = Z[v,:] . a_src and q[v] = Z[v,:] . a_dst (Z = the
// transformed embeddings), which the edge kernels combine per edge.  Forward: both dot products
// from one read of Z.  Backward (chain rule through the two products): the gradient of Z gains
// dp[v] a_src + dq[v] a_dst, and da_src = Z^T dp, da_dst = Z^T dq.
//
// Both are bound by memory (one read of Z forward; one of Z and dZ and one write of dZ backward), so rows are read in
// 16-byte vectors where their alignment allows (VEC = 4; else single floats), several rows in flight per thread.
// Forward: a group of L lanes per vertex (L x VEC covers the width up to 64 lanes), xor-tree sums.  Backward: a
// block owns a contiguous range of vertices; thread (ty, tx) walks the vertices ty, ty + TY, ... of the
// range for the vectors tx, tx + TX, ...; the column sums of a block are combined over ty in a fixed order through LDS and those
// of the blocks by a second kernel, 16 at a time in a fixed tree, so the result is deterministic.
// Measured (169,343 x 64): forward 0.026 -> 0.009 ms, backward 0.052 -> 0.023 ms, its second kernel (which added the partial
// sums of 512 blocks one after the other) 0.125 -> 0.006 ms.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lane_util.h"
#include "ntp_internal.h"

namespace ntp {

namespace {

constexpr int MAX_WIDTH = 1024;
constexpr int MAX_BLOCKS = 1024;                    // partial column sums kept per call, ...
constexpr int64_t MAX_SCRATCH = 4ll << 20;          // ... at most this many bytes of them

template <int VEC> __device__ __forceinline__ void load_cols(const float* p, float (&v)[VEC]) {
    if constexpr (VEC == 4) { const float4 t = *reinterpret_cast<const float4*>(p); v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w; }
    else v[0] = *p;
}
template <int VEC> __device__ __forceinline__ void store_cols(float* p, const float (&v)[VEC]) {
    if constexpr (VEC == 4) *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
    else *p = v[0];
}

template <int L, int VEC>
__global__ void __launch_bounds__(256) scores_fwd_kernel(const float* __restrict__ Z, const float* __restrict__ a_src,
                                                         const float* __restrict__ a_dst, float* __restrict__ p,
                                                         float* __restrict__ q, int64_t n, int m, int64_t ldz) {
    constexpr int R = 64 / L, U = 4;       // rows of a wavefront at a time, and in flight
    const int lane = threadIdx.x & 63;
    const int g = lane / L, l = lane % L;
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * (R * U) + g;
    float sp[U], sq[U];
#pragma unroll
    for (int u = 0; u < U; ++u) sp[u] = sq[u] = 0.f;
    for (int j = l * VEC; j < m; j += L * VEC) {
        float x[U][VEC], as[VEC], ad[VEC];
        load_cols<VEC>(a_src + j, as);
        load_cols<VEC>(a_dst + j, ad);
#pragma unroll
        for (int u = 0; u < U; ++u) load_cols<VEC>(Z + (row0 + u * R < n ? row0 + u * R : 0) * ldz + j, x[u]);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                sp[u] = fmaf(x[u][i], as[i], sp[u]);
                sq[u] = fmaf(x[u][i], ad[i], sq[u]);
            }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float s = group_sum<L>(sp[u], lane), d = group_sum<L>(sq[u], lane);
        if (row0 + u * R < n && l == 0) { p[row0 + u * R] = s; q[row0 + u * R] = d; }
    }
}

// TX vectors x TY vertices per block step, TX * TY = 256; NC vectors per thread
template <int TX, int VEC, int NC>
__global__ void __launch_bounds__(256) scores_bwd_kernel(const float* __restrict__ Z, const float* __restrict__ a_src,
                                                         const float* __restrict__ a_dst, const float* __restrict__ dp,
                                                         const float* __restrict__ dq, float* __restrict__ dZ,
                                                         float* __restrict__ partial, int64_t n, int m, int64_t ldz,
                                                         int64_t lddz, int64_t rows_per_block) {
    constexpr int TY = 256 / TX, U = NC == 1 ? 4 : 1;          // rows in flight
    __shared__ float red[256];
    const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
    const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
    const int64_t r1 = r0 + rows_per_block < n ? r0 + rows_per_block : n;
    float as[NC][VEC], ad[NC][VEC], acc_s[NC][VEC], acc_d[NC][VEC];
    bool on[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const int c = (tx + j * TX) * VEC;
        on[j] = c < m;
#pragma unroll
        for (int i = 0; i < VEC; ++i) as[j][i] = ad[j][i] = acc_s[j][i] = acc_d[j][i] = 0.f;
        if (on[j]) { load_cols<VEC>(a_src + c, as[j]); load_cols<VEC>(a_dst + c, ad[j]); }
    }
    for (int64_t r = r0 + ty; r < r1; r += U * TY) {
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            if (!on[j]) continue;
            const int c = (tx + j * TX) * VEC;
            float z[U][VEC], g[U][VEC], gp[U], gq[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t ru = r + u * TY < r1 ? r + u * TY : r;
                gp[u] = dp[ru];
                gq[u] = dq[ru];
                load_cols<VEC>(Z + ru * ldz + c, z[u]);
                load_cols<VEC>(dZ + ru * lddz + c, g[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (r + u * TY >= r1) break;
#pragma unroll
                for (int i = 0; i < VEC; ++i) {
                    g[u][i] += gp[u] * as[j][i] + gq[u] * ad[j][i];
                    acc_s[j][i] = fmaf(z[u][i], gp[u], acc_s[j][i]);
                    acc_d[j][i] = fmaf(z[u][i], gq[u], acc_d[j][i]);
                }
                store_cols<VEC>(dZ + (r + u * TY) * lddz + c, g[u]);
            }
        }
    }
    // column sums of the block: over ty in order, one column and one vector at a time
    float* out = partial + (int64_t)blockIdx.x * 2 * m;
#pragma unroll
    for (int j = 0; j < NC; ++j)
#pragma unroll
        for (int i = 0; i < VEC; ++i)
#pragma unroll
            for (int which = 0; which < 2; ++which) {
                red[threadIdx.x] = which ? acc_d[j][i] : acc_s[j][i];
                __syncthreads();
                const int c = (tx + j * TX) * VEC + i;
                if (ty == 0 && c < m) {
                    float s = 0.f;
                    for (int y = 0; y < TY; ++y) s += red[y * TX + tx];
                    out[which * m + c] = s;
                }
                __syncthreads();
            }
}

// 16 columns of (da_src, da_dst) per block; thread (ty, tx) adds the blocks ty, ty + 16, ... of column tx in order
__global__ void __launch_bounds__(256) scores_bwd_final_kernel(const float* __restrict__ partial, float* __restrict__ da_src,
                                                               float* __restrict__ da_dst, int m, int n_blocks) {
    __shared__ float red[16][17];
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    const int c = blockIdx.x * 16 + tx;
    float s = 0.f;
    if (c < 2 * m) {
        const float* p = partial + c;
        int b = ty;
        for (; b + 48 < n_blocks; b += 64) {             // four loads in flight
            float t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] = p[(int64_t)(b + 16 * u) * 2 * m];
#pragma unroll
            for (int u = 0; u < 4; ++u) s += t[u];
        }
        for (; b < n_blocks; b += 16) s += p[(int64_t)b * 2 * m];
    }
    red[ty][tx] = s;
    __syncthreads();
    if (ty == 0 && c < 2 * m) {
        float r = 0.f;
#pragma unroll
        for (int y = 0; y < 16; ++y) r += red[y][tx];
        if (c < m) da_src[c] = r;
        else da_dst[c - m] = r;
    }
}

int bwd_blocks(int64_t n, int64_t m) {
    // about 16 rows per thread of a 64-column matrix (16 vectors x 16 rows per step), at most four blocks per compute unit
    const int64_t rows = std::max<int64_t>(16, 16384 / std::max<int64_t>(16, m));
    const int64_t most = std::min<int64_t>(MAX_BLOCKS, MAX_SCRATCH / (2 * m * (int64_t)sizeof(float)));
    return (int)std::max<int64_t>(1, std::min<int64_t>((n + rows - 1) / rows, most));
}

}  // namespace

int64_t attention_scores_max_width() { return MAX_WIDTH; }

int64_t attention_scores_bwd_scratch_bytes(int64_t n, int64_t m) {
    if (n <= 0 || m <= 0) return 0;
    return (int64_t)bwd_blocks(n, m) * 2 * m * (int64_t)sizeof(float);
}

int launch_attention_scores_fwd(const float* Z, const float* a_src, const float* a_dst, float* p, float* q,
                                int64_t n, int64_t m, int64_t ldz, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    const bool vec4 = m % 4 == 0 && ldz % 4 == 0 && (uintptr_t)Z % 16 == 0 && (uintptr_t)a_src % 16 == 0 && (uintptr_t)a_dst % 16 == 0;
    const int64_t nv = vec4 ? m / 4 : m;
    int L = 4;
    while (L < 64 && L < nv) L <<= 1;
    const int64_t rows_per_block = 4 * (64 / L) * 4;
    const dim3 grid((unsigned)((n + rows_per_block - 1) / rows_per_block));
#define NTP_SCORES_FWD(LL)                                                                                                                  \
    do {                                                                                                                                    \
        if (vec4) hipLaunchKernelGGL((scores_fwd_kernel<LL, 4>), grid, dim3(256), 0, st, Z, a_src, a_dst, p, q, n, (int)m, ldz);             \
        else hipLaunchKernelGGL((scores_fwd_kernel<LL, 1>), grid, dim3(256), 0, st, Z, a_src, a_dst, p, q, n, (int)m, ldz);                  \
    } while (0)
    switch (L) {
        case 4: NTP_SCORES_FWD(4); break;
        case 8: NTP_SCORES_FWD(8); break;
        case 16: NTP_SCORES_FWD(16); break;
        case 32: NTP_SCORES_FWD(32); break;
        default: NTP_SCORES_FWD(64); break;
    }
#undef NTP_SCORES_FWD
    if (hipGetLastError() != hipSuccess) { set_error("attention score kernel launch failed"); return NTP_EHIP; }
    return NTP_OK;
}

int launch_attention_scores_bwd(const float* Z, const float* a_src, const float* a_dst, const float* dp, const float* dq,
                                float* dZ, float* da_src, float* da_dst, int64_t n, int64_t m, int64_t ldz, int64_t lddz,
                                float* scratch, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    const int nb = bwd_blocks(n, m);
    const int64_t rows_per_block = (n + nb - 1) / nb;
    const bool vec4 = m % 4 == 0 && ldz % 4 == 0 && lddz % 4 == 0 && (uintptr_t)Z % 16 == 0 && (uintptr_t)dZ % 16 == 0 &&
                      (uintptr_t)a_src % 16 == 0 && (uintptr_t)a_dst % 16 == 0;
    const int64_t nv = vec4 ? m / 4 : m;
    int tx = 4;
    while (tx < 256 && tx < nv) tx <<= 1;
#define NTP_SCORES_BWD(TX, VEC, NC) hipLaunchKernelGGL((scores_bwd_kernel<TX, VEC, NC>), dim3((unsigned)nb), dim3(256), 0, st, Z, a_src, a_dst, dp, dq, dZ, \
                                              scratch, n, (int)m, ldz, lddz, rows_per_block)
    if (vec4) {
        switch (tx) {
            case 4: NTP_SCORES_BWD(4, 4, 1); break;
            case 8: NTP_SCORES_BWD(8, 4, 1); break;
            case 16: NTP_SCORES_BWD(16, 4, 1); break;
            case 32: NTP_SCORES_BWD(32, 4, 1); break;
            case 64: NTP_SCORES_BWD(64, 4, 1); break;
            case 128: NTP_SCORES_BWD(128, 4, 1); break;
            default: NTP_SCORES_BWD(256, 4, 1); break;
        }
    } else {
        switch (tx) {
            case 4: NTP_SCORES_BWD(4, 1, 1); break;
            case 8: NTP_SCORES_BWD(8, 1, 1); break;
            case 16: NTP_SCORES_BWD(16, 1, 1); break;
            case 32: NTP_SCORES_BWD(32, 1, 1); break;
            case 64: NTP_SCORES_BWD(64, 1, 1); break;
            case 128: NTP_SCORES_BWD(128, 1, 1); break;
            default: NTP_SCORES_BWD(256, 1, 4); break;
        }
    }
#undef NTP_SCORES_BWD
    hipLaunchKernelGGL(scores_bwd_final_kernel, dim3((unsigned)((2 * m + 15) / 16)), dim3(256), 0, st, scratch, da_src, da_dst, (int)m, nb);
    if (hipGetLastError() != hipSuccess) { set_error("attention score gradient kernel launch failed"); return NTP_EHIP; }
    return NTP_OK;
}

}  // namespace ntp
