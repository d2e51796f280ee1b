// Edge attention weights of GAT-style aggregation (AGG of GAT, Section 2.1 of the paper;
// Section 4.1 computes them for all edges before the aggregation starts):
//   e(u -> v) = LeakyReLU(p[u] + q[v]),   alpha(u -> v) = exp(e(u -> v)) / sum over the
//   in-edges (u' -> v) of exp(e(u' -> v))
// with per-vertex scores p (source half of the mapping a^T [. || .]) and q (destination half).
//
// Rows of the by-destination form are softmax rows: a lane group (rows of up to 8 or 32
// entries) or a wavefront (longer rows) takes the row maximum, the sum of exponentials and
// writes the weights; rows beyond the split threshold go segment by segment (one block each,
// partial maxima and sums combined per row); all reductions in fixed trees
// (deterministic).  The score q, the maximum and the reciprocal sum of every destination are
// kept, so the same weights can be written in the entry order of the by-source form element
// by element, with the same arithmetic (bit-identical numbers for an edge in both orders).
#include <hip/hip_runtime.h>

#include <cmath>

#include "lane_util.h"
#include "ntp_internal.h"

namespace ntp {

namespace {

__device__ __forceinline__ float lrelu(float x, float slope) { return x > 0.f ? x : slope * x; }

// Per destination v the by-destination pass leaves st[v] = (q[v], row maximum, 1 / row sum, 0):
// one 16-byte gather gives the by-source pass everything it needs about v.
//
// alpha = exp(e - maximum) * (1 / sum) in both passes, from the same stored numbers.
__device__ __forceinline__ float weight_of(float e, float mx, float rs) { return expf(e - mx) * rs; }

// One group of L lanes per row; rows taken from rows[0..n_rows).
// TRANSPOSED = false: rows are destinations v, columns sources u; writes alpha and st[v].
// TRANSPOSED = true : rows are sources u, columns destinations v; reads st[v].
// Entries are taken four per lane at a time so that four gathers are in flight.  A row longer
// than 4 L entries parks its scores in the output array after the first sweep, so the random
// gathers of p happen once and the later sweeps read consecutive memory.
template <int L, bool TRANSPOSED>
__device__ __forceinline__ void attention_rows(const AttArgs& a, int block, int first, int n_rows) {
    constexpr int R = 64 / L;
    const int lane = threadIdx.x & 63;
    const int g = lane / L, l = lane % L;
    const int64_t idx = ((int64_t)block * 4 + (threadIdx.x >> 6)) * R + g;
    const bool valid = idx < n_rows;
    int row = 0;
    int64_t beg = 0;
    int64_t d = 0;
    if (valid) {
        row = a.rows[first + idx];
        beg = a.rowptr[row];
        d = a.rowptr[row + 1] - beg;
    }
    const int32_t* ci = a.colidx + beg;
    float* out = a.alpha + beg;
    if constexpr (TRANSPOSED) {
        const float pu = valid ? a.p[row] : 0.f;
        for (int64_t k0 = l; k0 < d; k0 += 4 * L) {
            int c[4];
            float4 t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) c[u] = k0 + u * L < d ? ci[k0 + u * L] : row;
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] = reinterpret_cast<const float4*>(a.st)[c[u]];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (k0 + u * L < d) out[k0 + u * L] = weight_of(lrelu(pu + t[u].x, a.slope), t[u].y, t[u].z);
        }
        return;
    }
    const float qv = valid ? a.q[row] : 0.f;
    // first sweep: scores of up to four entries per lane stay in registers
    float e[4];
    {
        int c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = l + u * L < d ? ci[l + u * L] : row;
#pragma unroll
        for (int u = 0; u < 4; ++u) e[u] = l + u * L < d ? lrelu(a.p[c[u]] + qv, a.slope) : -INFINITY;
    }
    float m = fmaxf(fmaxf(e[0], e[1]), fmaxf(e[2], e[3]));
    const bool longer = __ballot(d > 4 * L) != 0;          // some row of the wavefront needs more sweeps
    if (longer) {
        for (int64_t k0 = l + 4 * L; k0 < d; k0 += 4 * L) {
            int c[4];
            float x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) c[u] = k0 + u * L < d ? ci[k0 + u * L] : row;
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = lrelu(a.p[c[u]] + qv, a.slope);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (k0 + u * L < d) { out[k0 + u * L] = x[u]; m = fmaxf(m, x[u]); }
        }
    }
    m = group_max<L>(m, lane);
    float s = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) s += l + u * L < d ? expf(e[u] - m) : 0.f;
    if (longer)
        for (int64_t k = l + 4 * L; k < d; k += L) s += expf(out[k] - m);
    s = group_sum<L>(s, lane);
    const float rs = 1.f / s;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (l + u * L < d) out[l + u * L] = weight_of(e[u], m, rs);
    if (longer)
        for (int64_t k = l + 4 * L; k < d; k += L) out[k] = weight_of(out[k], m, rs);
    if (valid && l == 0) reinterpret_cast<float4*>(a.st)[row] = d > 0 ? make_float4(qv, m, rs, 0.f) : make_float4(qv, 0.f, 1.f, 0.f);
}

// ---- rows beyond the split threshold: one block per segment (the pieces the aggregation
// cuts such rows into), so that a hub row of 10^5 entries is spread over many blocks ---------
// pass 1: scores parked in the output array; per segment maximum and sum of exp(score - maximum)
__device__ __forceinline__ void attention_segment_stats(const AttArgs& a, const Segment& sg, float2* seg_stats) {
    __shared__ float red[4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int32_t* ci = a.colidx + sg.e_begin;
    float* out = a.alpha + sg.e_begin;
    const float qv = a.q[sg.row];
    float m = -INFINITY;
    for (int k = threadIdx.x; k < sg.len; k += 256) {
        const float x = lrelu(a.p[ci[k]] + qv, a.slope);
        out[k] = x;
        m = fmaxf(m, x);
    }
    m = group_max<64>(m, lane);
    if (lane == 0) red[w] = m;
    __syncthreads();
    m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();
    float s = 0.f;
    for (int k = threadIdx.x; k < sg.len; k += 256) s += expf(out[k] - m);
    s = group_sum<64>(s, lane);
    if (lane == 0) red[w] = s;
    __syncthreads();
    if (threadIdx.x == 0) seg_stats[sg.slot] = make_float2(m, (red[0] + red[1]) + (red[2] + red[3]));
}

// a wavefront combines the segments of a row: maximum of the maxima, sums rescaled to it and added in a fixed tree
__device__ __forceinline__ float2 attention_combine(const ReduceItem& it, const float2* seg_stats, int lane) {
    const float2* st = seg_stats + it.first_slot;
    float m = -INFINITY;
    for (int k = lane; k < it.n_slots; k += 64) m = fmaxf(m, st[k].x);
    m = group_max<64>(m, lane);
    float s = 0.f;
    for (int k = lane; k < it.n_slots; k += 64) s += st[k].y * expf(st[k].x - m);
    s = group_sum<64>(s, lane);
    return make_float2(m, 1.f / s);
}
// pass 2 where the segments do not do it: one wavefront per split row
__global__ void __launch_bounds__(64) attention_combine_kernel(const AttArgs a, const ReduceItem* items, const float2* seg_stats) {
    const ReduceItem it = items[blockIdx.x];
    const float2 t = attention_combine(it, seg_stats, threadIdx.x);
    if (threadIdx.x == 0) reinterpret_cast<float4*>(a.st)[it.row] = make_float4(a.q[it.row], t.x, t.y, 0.f);
}

// pass 3 (by destination): parked scores -> weights.  items: pass 2 as well, by every wavefront of the row's segments for itself (a
// launch less, 5 us)
__global__ void __launch_bounds__(256) attention_segment_write_kernel(const AttArgs a, const Segment* segs, const ReduceItem* items, const float2* seg_stats) {
    const Segment sg = segs[blockIdx.x];
    float* out = a.alpha + sg.e_begin;
    float2 t;
    if (items) {
        const ReduceItem it = items[sg.item];
        t = attention_combine(it, seg_stats, threadIdx.x & 63);
        if (sg.slot == it.first_slot && threadIdx.x == 0) reinterpret_cast<float4*>(a.st)[sg.row] = make_float4(a.q[sg.row], t.x, t.y, 0.f);
    } else {
        const float4 st = reinterpret_cast<const float4*>(a.st)[sg.row];
        t = make_float2(st.y, st.z);
    }
    for (int k = threadIdx.x; k < sg.len; k += 256) out[k] = weight_of(out[k], t.x, t.y);
}
// by source: the element-wise form
__device__ __forceinline__ void attention_segment_write_transposed(const AttArgs& a, const Segment& sg) {
    float* out = a.alpha + sg.e_begin;
    const int32_t* ci = a.colidx + sg.e_begin;
    const float pu = a.p[sg.row];
    for (int k = threadIdx.x; k < sg.len; k += 256) {
        const float4 t = reinterpret_cast<const float4*>(a.st)[ci[k]];
        out[k] = weight_of(lrelu(pu + t.x, a.slope), t.y, t.z);
    }
}

// Everything that depends on nothing else in one launch, long rows first (they are the longest-running pieces): blocks
// [0, n_segs) take the segments of split rows, the next ones the rows of more than 32, more than 8 and
// up to 8 entries (64, 32 and 8 lanes each).
struct AttRanges {
    const Segment* segs;
    int n_segs;
    int first[3], count[3];
    int block_end[3];          // first block after each range of rows
};
template <bool TRANSPOSED>
__global__ void __launch_bounds__(256) attention_kernel(const AttArgs a, const AttRanges r, float2* seg_stats) {
    const int b = (int)blockIdx.x;
    if (b < r.n_segs) {
        if constexpr (TRANSPOSED) attention_segment_write_transposed(a, r.segs[b]);
        else attention_segment_stats(a, r.segs[b], seg_stats);
    } else if (b < r.block_end[0]) {
        attention_rows<64, TRANSPOSED>(a, b - r.n_segs, r.first[0], r.count[0]);
    } else if (b < r.block_end[1]) {
        attention_rows<32, TRANSPOSED>(a, b - r.block_end[0], r.first[1], r.count[1]);
    } else {
        attention_rows<8, TRANSPOSED>(a, b - r.block_end[1], r.first[2], r.count[2]);
    }
}

// ---- gradient of the scores through the attention weights --------------------------------------
// Given dY = dLoss/dY of Y[v,:] = sum_u alpha(u -> v) Z[u,:]:
//   dalpha(u -> v) = dY[v,:] . Z[u,:],  t[v] = sum_u alpha dalpha,  de = alpha (dalpha - t[v]),
//   ds = de * (1 if p[u] + q[v] > 0 else slope),  dq[v] = sum over in-edges of ds,
//   dp[u] = sum over out-edges of ds.
// By-destination pass (rows v, own = dY[v,:], gathered = Z[u,:]): dalpha of every entry (parked in
// scratch), t[v], dq[v].  By-source pass (rows u, own = Z[u,:], gathered = dY[v,:]): dalpha again
// in that order, with t[v] and alpha in by-source order: dp[u].  A group of L lanes (4, 8 or 16) forms one dot
// product at a time (L x VEC x NJ columns, xor tree over the group) and takes its entries L at a time: lane l loads id and
// weight of the l-th (one coalesced load each, where one broadcast load per entry used to take as many issue slots as
// the gathers), the ids are handed round inside the group, and lane l keeps the l-th dot product, so that weights, gates
// and parked values are again one coalesced access per L entries.  Rows of more than 128 entries take one block (its
// groups share the entries, partial sums combined through LDS in a fixed order; one wavefront per such row measured
// slower); rows beyond the split threshold one block per segment, the partial sums of the segments combined by a small
// kernel in segment order.  Where both sweeps run in one kernel a lane keeps its first entry in
// registers (short rows park nothing) and a parked dalpha is read back by the thread that wrote it.
// Widest row: 1024 columns with 16-byte vectors, 256 otherwise.
// Measured (169,343 vertices, 2.5 M entries, 64 columns, by destination): 0.178 -> 0.114 ms for the whole pass.
template <int VEC, int NJ, int L>
struct DotRow {
    float own[NJ][VEC];
    int col[NJ];
    bool on[NJ];
    __device__ __forceinline__ void load_own(const float* row, int l, int m) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            col[j] = (j * L + l) * VEC;
            on[j] = col[j] < m;
#pragma unroll
            for (int i = 0; i < VEC; ++i) own[j][i] = 0.f;
            if (on[j]) {
                if constexpr (VEC == 4) { const float4 t = *reinterpret_cast<const float4*>(row + col[j]); own[j][0] = t.x; own[j][1] = t.y; own[j][2] = t.z; own[j][3] = t.w; }
                else own[j][0] = row[col[j]];
            }
        }
    }
    // this lane's share of own . other (columns outside the row contribute zero)
    __device__ __forceinline__ float partial(const float* other) const {
        float acc = 0.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            if (on[j]) {
                if constexpr (VEC == 4) {
                    const float4 t = *reinterpret_cast<const float4*>(other + col[j]);
                    acc = fmaf(own[j][0], t.x, acc); acc = fmaf(own[j][1], t.y, acc);
                    acc = fmaf(own[j][2], t.z, acc); acc = fmaf(own[j][3], t.w, acc);
                } else {
                    acc = fmaf(own[j][0], other[col[j]], acc);
                }
            }
        }
        return acc;
    }
};

template <int VEC, int NJ, int L, int U, int J, int I>
__device__ __forceinline__ void group_gathers(const DotRow<VEC, NJ, L>& dot, const float* other, int64_t ld, int c, int lane, float (&part)[U]) {
    if constexpr (I < U) {
        part[I] = dot.partial(other + (int64_t)group_bcast<L, J + I>(c, lane) * ld);
        group_gathers<VEC, NJ, L, U, J, I + 1>(dot, other, ld, c, lane, part);
    }
}
// the dot products of the group's entries J .. L-1 whose ids the lanes hold in c: lane j ends with that of entry j.  Entries
// from nb on (nb differs between the groups of a wavefront) are looked up in vain.
template <int VEC, int NJ, int L, int U, int J = 0>
__device__ __forceinline__ void group_dots(const DotRow<VEC, NJ, L>& dot, const float* other, int64_t ld, int c, int nb, int lane, float& da) {
    if constexpr (J < L) {
        if (__ballot(J < nb) == 0) return;
        float part[U];
        group_gathers<VEC, NJ, L, U, J, 0>(dot, other, ld, c, lane, part);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float s = group_sum<L>(part[u], lane);
            da = lane % L == J + u ? s : da;
        }
        group_dots<VEC, NJ, L, U, J + U>(dot, other, ld, c, nb, lane, da);
    }
}

// WORK_GROUP  : one row per group of L lanes, rows[first .. first + n_rows), `block` counts the blocks of this kind.
// WORK_BLOCK  : one row per block (its 256 / L groups take L entries each in turn), rows[first + block].
// WORK_SEG    : one segment of a split row per block, segs[block]: the dot products of its
//               entries; the partial t (by destination) or partial dp (by source) goes to the
//               segment's slot.
enum { WORK_GROUP = 0, WORK_BLOCK = 1, WORK_SEG = 2 };

// sum over the NG groups of a block of a value all lanes of a group hold, in a fixed order
template <int L>
__device__ __forceinline__ float block_sum(float v, float* red) {
    constexpr int NG = 256 / L;
    if (threadIdx.x % L == 0) red[threadIdx.x / L] = v;
    __syncthreads();
    float s = 0.f;
    for (int i = 0; i < NG; ++i) s += red[i];
    __syncthreads();
    return s;
}

template <int VEC, int NJ, int L, bool TRANSPOSED, int WORK>
__device__ __forceinline__ void attention_bwd_work(const AttBwdArgs& a, int block, int first, int n_rows, const Segment* segs, float* red) {
    constexpr bool SEG = WORK == WORK_SEG;
    constexpr int R = 64 / L;                                          // groups per wavefront
    constexpr int SHARE = WORK == WORK_GROUP ? 1 : 256 / L;            // groups on one row
    constexpr int U = NJ == 1 ? (L < 8 ? L : 8) : 4;                   // dot products in flight per group
    const int lane = threadIdx.x & 63;
    const int l = lane % L;
    const int gi = SHARE == 1 ? 0 : (int)(threadIdx.x / L);            // group among those on the row
    int row = 0;
    int slot = 0;
    bool valid = true;
    int64_t beg = 0;
    int d = 0;
    if constexpr (SEG) {
        const Segment sg = segs[block];
        row = sg.row; slot = sg.slot; beg = sg.e_begin; d = sg.len;
    } else {
        const int64_t idx = WORK == WORK_BLOCK ? (int64_t)block : ((int64_t)block * 4 + (threadIdx.x >> 6)) * R + lane / L;
        valid = idx < n_rows;
        if (valid) { row = a.rows[first + idx]; beg = a.rowptr[row]; d = (int)(a.rowptr[row + 1] - beg); }
    }
    const int32_t* ci = a.colidx + beg;
    const float* al = a.alpha + beg;
    float* park = a.park + beg;
    auto share_sum = [&](float v) {
        if constexpr (SHARE == 1) return v;
        else return block_sum<L>(v, red);
    };
    const bool writer = SHARE == 1 ? valid && l == 0 : threadIdx.x == 0;
    DotRow<VEC, NJ, L> dot;
    dot.load_own(a.own + (int64_t)row * a.ld_own, l, valid ? a.m : 0);
    // this lane's entry of the group's batch at k: column id and weight (an entry that does not exist: the row's own vertex, 0)
    auto entry = [&](int k, int& c, float& w) {
        c = row;
        w = 0.f;
        if (k + l < d) { c = ci[k + l]; w = al[k + l]; }
    };
    const float own_pq = valid ? (TRANSPOSED ? a.p[row] : a.q[row]) : 0.f;
    int c, c0;
    float w, w0;
    int k = gi * L;
    entry(k, c, w);
    c0 = c;
    w0 = w;
    float sum = 0.f, da0 = 0.f;
    for (; __ballot(k < d) != 0; k += SHARE * L) {                     // the wavefront stays together for the shuffles
        int cn;
        float wn;
        entry(k + SHARE * L, cn, wn);                                   // the next batch is fetched meanwhile
        float da = 0.f;
        group_dots<VEC, NJ, L, U>(dot, a.other, a.ld_other, c, d - k, lane, da);
        const bool in = k + l < d;
        if constexpr (TRANSPOSED) {
            if (in) {
                const float2 tq = reinterpret_cast<const float2*>(a.t)[c];      // (t, q) of the destination
                sum += w * (da - tq.x) * (own_pq + tq.y > 0.f ? 1.f : a.slope);
            }
        } else {
            if (in) {
                sum += w * da;
                if (SEG || k >= SHARE * L) park[k + l] = da;
                else da0 = da;                                          // the first entry stays in a register
            }
        }
        c = cn;
        w = wn;
    }
    sum = share_sum(group_sum<L>(sum, lane));
    if constexpr (SEG) {
        if (writer) a.slots[slot] = sum;
    } else if constexpr (TRANSPOSED) {
        if (writer) a.out[row] = a.accumulate ? a.out[row] + sum : sum;
    } else {
        // sum = t: ds of the entries of this lane, added over the row
        const float t = sum;
        float dqp = 0.f;
        for (int e = gi * L + l; e < d; e += SHARE * L) {
            const bool kept = e < SHARE * L;
            const int cc = kept ? c0 : ci[e];
            const float wv = ((kept ? da0 : park[e]) - t) * (a.p[cc] + own_pq > 0.f ? 1.f : a.slope);
            if (a.keep_w) park[e] = wv;
            dqp += (kept ? w0 : al[e]) * wv;
        }
        dqp = share_sum(group_sum<L>(dqp, lane));
        if (writer) { a.out[row] = a.accumulate ? a.out[row] + dqp : dqp; reinterpret_cast<float2*>(a.t)[row] = make_float2(t, own_pq); }
    }
}

// out[row] = sum of the row's slots, in segment order
__device__ __forceinline__ float slots_sum(const ReduceItem& it, const float* slots) {
    float s = 0.f;
    for (int j = 0; j < it.n_slots; ++j) s += slots[it.first_slot + j];
    return s;
}
__device__ __forceinline__ void attention_combine_slots(const AttCombine& c, int block) {
    const int i = block * 256 + threadIdx.x;
    if (i >= c.n_items) return;
    const ReduceItem it = c.items[i];
    const float s = slots_sum(it, c.slots);
    c.out[it.row] = c.accumulate ? c.out[it.row] + s : s;
}

// blocks [0, n_segs): the segments of split rows; the next n_block_rows: rows of more than 128 entries; then the rest, and at the
// end (by source) what is left of dq
template <int VEC, int NJ, int L, bool TRANSPOSED>
__global__ void __launch_bounds__(256) attention_bwd_kernel(const AttBwdArgs a, int n_segs, const Segment* segs, int n_group_rows, int n_block_rows,
                                                            const AttCombine also, int also_first) {
    __shared__ float red[256 / L];
    const int b = (int)blockIdx.x;
    if (TRANSPOSED && b >= also_first) { attention_combine_slots(also, b - also_first); return; }
    if (b < n_segs) attention_bwd_work<VEC, NJ, L, TRANSPOSED, WORK_SEG>(a, b, 0, 0, segs, red);
    else if (b < n_segs + n_block_rows) attention_bwd_work<VEC, NJ, L, TRANSPOSED, WORK_BLOCK>(a, b - n_segs, n_group_rows, n_block_rows, segs, red);
    else attention_bwd_work<VEC, NJ, L, TRANSPOSED, WORK_GROUP>(a, b - n_segs - n_block_rows, 0, n_group_rows, segs, red);
}

// by destination, after the slots of t: ds of a segment's entries from the parked dalpha, partial dq to its slot.  items: t is summed
// here, by every block of the row for itself (a launch less); else it is in place
__global__ void __launch_bounds__(256) attention_bwd_segment_ds_kernel(const AttBwdArgs a, const Segment* segs, const ReduceItem* items) {
    __shared__ float red[4];
    const Segment sg = segs[blockIdx.x];
    const int32_t* ci = a.colidx + sg.e_begin;
    const float* al = a.alpha + sg.e_begin;
    float* park = a.park + sg.e_begin;
    const float qv = a.q[sg.row];
    float t;
    if (items) {
        const ReduceItem it = items[sg.item];
        t = slots_sum(it, a.slots);
        if (sg.slot == it.first_slot && threadIdx.x == 0) reinterpret_cast<float2*>(a.t)[sg.row] = make_float2(t, qv);
    } else {
        t = a.t[2 * sg.row];
    }
    float dqp = 0.f;
    for (int k = threadIdx.x; k < sg.len; k += 256) {
        const float wv = (park[k] - t) * (a.p[ci[k]] + qv > 0.f ? 1.f : a.slope);
        if (a.keep_w) park[k] = wv;
        dqp += al[k] * wv;
    }
    dqp = block_sum<64>(group_sum<64>(dqp, threadIdx.x & 63), red);
    if (threadIdx.x == 0) a.dq_slots[sg.slot] = dqp;
}

// dp[u] = sum over the by-source entries k of row u of alpha[k] * w[perm[k]] (EDGE_PERM graphs: w of every edge sits in
// by-destination order).  One scalar per entry, so the lanes of a group take entries and not columns: blocks
// [0, n_segs) the segments of split rows (to the slots), then 64 lanes for the rows of more than 32 entries, 8 for the others.
template <int L>
__device__ __forceinline__ void perm_sum_rows(const AttBwdArgs& a, const int32_t* perm, int block, int first, int n_rows) {
    constexpr int R = 64 / L;
    const int lane = threadIdx.x & 63, l = lane % L;
    const int64_t idx = ((int64_t)block * 4 + (threadIdx.x >> 6)) * R + lane / L;
    if (idx - lane / L >= n_rows) return;                  // the whole wavefront
    const bool valid = idx < n_rows;
    int row = 0;
    int64_t beg = 0;
    int d = 0;
    if (valid) { row = a.rows[first + idx]; beg = a.rowptr[row]; d = (int)(a.rowptr[row + 1] - beg); }
    float s = 0.f;
    for (int k = l; k < d; k += 4 * L) {
        int c[4];
        float w[4], x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool in = k + u * L < d;
            c[u] = in ? perm[beg + k + u * L] : perm[beg];
            w[u] = in ? a.alpha[beg + k + u * L] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = a.park[c[u]];
#pragma unroll
        for (int u = 0; u < 4; ++u) s += k + u * L < d ? w[u] * x[u] : 0.f;
    }
    s = group_sum<L>(s, lane);
    if (valid && l == 0) a.out[row] = a.accumulate ? a.out[row] + s : s;
}

__global__ void __launch_bounds__(256) perm_sum_kernel(const AttBwdArgs a, const int32_t* perm, int n_segs, const Segment* segs,
                                                       int n_short_rows, int n_long_rows, const AttCombine also, int also_first) {
    __shared__ float red[4];
    const int b = (int)blockIdx.x, long_blocks = (n_long_rows + 3) / 4;
    if (b >= also_first) {
        attention_combine_slots(also, b - also_first);
    } else if (b < n_segs) {
        const Segment sg = segs[b];
        float s = 0.f;
        for (int k = threadIdx.x; k < sg.len; k += 256) s += a.alpha[sg.e_begin + k] * a.park[perm[sg.e_begin + k]];
        s = block_sum<64>(group_sum<64>(s, threadIdx.x & 63), red);
        if (threadIdx.x == 0) a.slots[sg.slot] = s;
    } else if (b < n_segs + long_blocks) {
        perm_sum_rows<64>(a, perm, b - n_segs, n_short_rows, n_long_rows);
    } else {
        perm_sum_rows<8>(a, perm, b - n_segs - long_blocks, 0, n_short_rows);
    }
}

__global__ void __launch_bounds__(256) attention_bwd_combine_kernel(const AttCombine c) { attention_combine_slots(c, (int)blockIdx.x); }

// (t, q) of the split rows where the segments do not sum t
__global__ void __launch_bounds__(256) attention_bwd_combine_t_kernel(const ReduceItem* items, int n_items, const float* slots, float* t, const float* q) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n_items) return;
    const ReduceItem it = items[i];
    reinterpret_cast<float2*>(t)[it.row] = make_float2(slots_sum(it, slots), q[it.row]);
}

template <int VEC, int NJ, int L, bool T>
int launch_bwd_shape(const AttBwdArgs& a, const AttBwdRows& r, hipStream_t st) {
    constexpr int ROWS_PER_BLOCK = 4 * (64 / L);
    const int64_t rows = (int64_t)r.n_segs + r.n_block_rows + (r.n_group_rows + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK;
    const int64_t blocks = rows + (r.also.n_items + 255) / 256;
    if (blocks == 0) return NTP_OK;
    hipLaunchKernelGGL((attention_bwd_kernel<VEC, NJ, L, T>), dim3((unsigned)blocks), dim3(256), 0, st, a, r.n_segs, r.segs,
                       r.n_group_rows, r.n_block_rows, r.also, (int)rows);
    return hipGetLastError() == hipSuccess ? NTP_OK : NTP_EHIP;
}

// lanes per group: the smallest of 4, 8, 16 whose vectors cover the row; wider rows take several
// vectors per lane
template <int VEC, bool T>
int launch_bwd_vec(const AttBwdArgs& a, const AttBwdRows& r, hipStream_t st) {
    const int nvec = (a.m + VEC - 1) / VEC;
    if (nvec <= 4) return launch_bwd_shape<VEC, 1, 4, T>(a, r, st);
    if (nvec <= 8) return launch_bwd_shape<VEC, 1, 8, T>(a, r, st);
    const int nj = (nvec + 15) / 16;
    if (nj <= 1) return launch_bwd_shape<VEC, 1, 16, T>(a, r, st);
    if (nj <= 2) return launch_bwd_shape<VEC, 2, 16, T>(a, r, st);
    if (nj <= 4) return launch_bwd_shape<VEC, 4, 16, T>(a, r, st);
    if (nj <= 8) return launch_bwd_shape<VEC, 8, 16, T>(a, r, st);
    if (nj <= 16) return launch_bwd_shape<VEC, 16, 16, T>(a, r, st);
    set_error("feature width %d too large for the attention gradient (at most %d)", a.m, 256 * VEC);
    return NTP_EUNSUPPORTED;
}

}  // namespace

// One chunk of a form, one phase at a time (a row beyond the split threshold may have its
// segments in several chunks, so the caller runs a phase over all chunks before the next):
//   phase 0: by destination: weights of all rows but the split ones, statistics of the split rows' segments;
//            by source: all weights
//   phase 1: per-row combination of the segment statistics (by-destination pass only)
//   phase 2: weights of the split rows' segments (by-destination pass only)
// combined: phase 2 does the work of phase 1 and that is left out (Plan::segments_combine)
// bins: bin_row_off / bin_count describe rows[] (see Plan); bins 0..3 hold rows of up to 8
// entries, 4..5 up to 32, the rest up to the split threshold; split rows come as segments
// (segs, n_segs), their rows as reduce items; seg_stats: two floats per partial-sum slot.
int launch_attention(const AttArgs& a, const int32_t* bin_row_off, const int32_t* bin_count,
                     const Segment* segs, int n_segs, const ReduceItem* split_rows, int n_split_rows,
                     float* seg_stats, bool transposed, int phase, bool combined, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    float2* ss = reinterpret_cast<float2*>(seg_stats);
    if (phase == 1) {
        if (!transposed && n_split_rows > 0)
            hipLaunchKernelGGL(attention_combine_kernel, dim3((unsigned)n_split_rows), dim3(64), 0, st, a, split_rows, ss);
    } else if (phase == 2) {
        if (!transposed && n_segs > 0)
            hipLaunchKernelGGL(attention_segment_write_kernel, dim3((unsigned)n_segs), dim3(256), 0, st, a, segs, combined ? split_rows : nullptr, ss);
    } else {
        AttRanges r;
        r.segs = segs;
        r.n_segs = n_segs;
        int end = n_segs;
        const int b0[3] = {6, 4, 0}, b1[3] = {NBINS - 1, 5, 3}, rows_per_block[3] = {4, 8, 32};
        for (int i = 0; i < 3; ++i) {
            r.first[i] = bin_row_off[b0[i]];
            r.count[i] = 0;
            for (int b = b0[i]; b <= b1[i]; ++b) r.count[i] += bin_count[b];
            end += (r.count[i] + rows_per_block[i] - 1) / rows_per_block[i];
            r.block_end[i] = end;
        }
        if (end > 0) {
            if (transposed) hipLaunchKernelGGL(attention_kernel<true>, dim3((unsigned)end), dim3(256), 0, st, a, r, ss);
            else hipLaunchKernelGGL(attention_kernel<false>, dim3((unsigned)end), dim3(256), 0, st, a, r, ss);
        }
    }
    if (hipGetLastError() != hipSuccess) { set_error("attention kernel launch failed"); return NTP_EHIP; }
    return NTP_OK;
}

// By destination: phase 0 = whole rows (dq, t) and the first sweep of the segments (partial t),
// 1 = t of the split rows from their slots, 2 = second sweep of the segments (partial dq),
// 3 = dq of the split rows.  By source: phase 0 = whole rows and segments (partial dp), 1 = dp of
// the split rows.  The caller runs each phase over every chunk before the next one.  combined: phase 2 does the work of phase 1 by
// destination, which is left out (as above); r.also: phase 0 by source does that of phase 3.  Each launch less is 5 us, the epoch of
// 2.5 M entries 1,420 -> 1,400 us.
// perm (by source only, nullable): the edge permutation, with w of every edge in a.park (see perm_sum_kernel).
int launch_attention_bwd(const AttBwdArgs& a, const AttBwdRows& r, bool transposed, int phase, bool combined, const int32_t* perm, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    int rc = NTP_OK;
    if (phase == 1 || phase == 3) {
        if (r.n_split_rows == 0) return NTP_OK;
        const dim3 blocks((unsigned)((r.n_split_rows + 255) / 256));
        if (phase == 1 && !transposed)
            hipLaunchKernelGGL(attention_bwd_combine_t_kernel, blocks, dim3(256), 0, st, r.split_rows, r.n_split_rows, a.slots, a.t, a.q);
        else
            hipLaunchKernelGGL(attention_bwd_combine_kernel, blocks, dim3(256), 0, st,
                               AttCombine{r.split_rows, transposed ? a.slots : a.dq_slots, a.out, r.n_split_rows, a.accumulate});
    } else if (phase == 2) {
        if (r.n_segs > 0)
            hipLaunchKernelGGL(attention_bwd_segment_ds_kernel, dim3((unsigned)r.n_segs), dim3(256), 0, st, a, r.segs, combined ? r.split_rows : nullptr);
    } else if (perm) {
        const int n_long = r.n_group_rows + r.n_block_rows - r.n_rows_32;
        const int64_t rows = (int64_t)r.n_segs + (n_long + 3) / 4 + (r.n_rows_32 + 31) / 32, blocks = rows + (r.also.n_items + 255) / 256;
        if (blocks > 0)
            hipLaunchKernelGGL(perm_sum_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a, perm, r.n_segs, r.segs, r.n_rows_32, n_long, r.also, (int)rows);
    } else {
        const bool vec4 = a.m % 4 == 0 && a.ld_own % 4 == 0 && a.ld_other % 4 == 0 &&
                          (uintptr_t)a.own % 16 == 0 && (uintptr_t)a.other % 16 == 0;
        if (vec4) rc = transposed ? launch_bwd_vec<4, true>(a, r, st) : launch_bwd_vec<4, false>(a, r, st);
        else rc = transposed ? launch_bwd_vec<1, true>(a, r, st) : launch_bwd_vec<1, false>(a, r, st);
        if (rc == NTP_EUNSUPPORTED) return rc;
    }
    if (rc != NTP_OK || hipGetLastError() != hipSuccess) { set_error("attention gradient kernel launch failed"); return NTP_EHIP; }
    return NTP_OK;
}

}  // namespace ntp
