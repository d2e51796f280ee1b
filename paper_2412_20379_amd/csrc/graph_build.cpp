// Host-side construction of the per-worker topology: the normalised adjacency of
// Section 4.1.3 in both compressed forms (by destination for eq. 1/3, by source for the
// backward pass of Section 4.2.1).  Pure C++, no device code.
//
// Processing order (fixed, so that the result is reproducible bit for bit):
//   input edges in input order; reversed copies after all originals (SYMMETRISE);
//   input self loops dropped and the first of equal (src,dst) kept (DEDUP);
//   one (v,v) entry of weight 1 per vertex appended last (ADD_SELF_LOOPS);
//   rows sorted by neighbour id, stable.
#include "ntp_internal.h"

#include <sys/mman.h>

#include <algorithm>
#include <atomic>
#include <climits>
#include <cmath>
#include <condition_variable>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <exception>
#include <mutex>
#include <new>
#include <thread>
#include <type_traits>
#include <utility>

namespace ntp {

// ---------------------------------------------------------------------------------------
static thread_local char g_err[512] = "";

void set_error(const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
}
const char* last_error() { return g_err; }

int host_threads() {
    unsigned hc = std::thread::hardware_concurrency();
    int t = hc ? (int)hc : 4;
    if (const char* e = getenv("NTP_HOST_THREADS")) t = atoi(e);
    return std::max(1, std::min(t, 32));
}

void parallel_run(int n_threads, void (*fn)(int, int, void*), void* ctx) {
    if (n_threads <= 1) { fn(0, 1, ctx); return; }
    std::vector<std::thread> th;
    th.reserve(n_threads - 1);
    for (int t = 1; t < n_threads; ++t) th.emplace_back(fn, t, n_threads, ctx);
    fn(0, n_threads, ctx);
    for (auto& x : th) x.join();
}

namespace {

// Threads that stay for the whole of one build (starting and joining them for every one of its passes took 0.2 ms a pass:
// most of the build of a small graph).  run(f) calls f(t) for t = 0 .. n-1 and returns when all are done.
class Workers {
public:
    explicit Workers(int n) : n_(n) {
        for (int t = 1; t < n; ++t) threads_.emplace_back([this, t] { loop(t); });
    }
    ~Workers() {
        {
            std::lock_guard<std::mutex> l(mu_);
            stop_ = true;
            ++turn_;
        }
        go_.notify_all();
        for (auto& t : threads_) t.join();
    }
    int size() const { return n_; }
    template <class F> void run(F&& f) {
        if (n_ == 1) { f(0); return; }
        call_ = [](void* c, int t) { (*static_cast<std::remove_reference_t<F>*>(c))(t); };
        arg_ = &f;
        left_.store(n_ - 1, std::memory_order_relaxed);
        {
            std::lock_guard<std::mutex> l(mu_);
            ++turn_;
        }
        go_.notify_all();
        guarded(0);
        std::unique_lock<std::mutex> l(mu_);
        done_.wait(l, [this] { return left_.load(std::memory_order_acquire) == 0; });
        if (error_) std::rethrow_exception(std::exchange(error_, nullptr));
    }
    // f(i) for i = 0 .. count-1, handed out `grain` at a time
    template <class F> void each(int64_t count, int64_t grain, F&& f) {
        std::atomic<int64_t> next{0};
        run([&](int) {
            for (;;) {
                const int64_t i0 = next.fetch_add(grain), i1 = std::min(count, i0 + grain);
                if (i0 >= count) break;
                for (int64_t i = i0; i < i1; ++i) f(i);
            }
        });
    }

private:
    void guarded(int t) {            // an exception (out of memory) surfaces in run()
        try {
            call_(arg_, t);
        } catch (...) {
            std::lock_guard<std::mutex> l(mu_);
            if (!error_) error_ = std::current_exception();
        }
    }
    void loop(int t) {
        uint64_t seen = 0;
        for (;;) {
            {
                std::unique_lock<std::mutex> l(mu_);
                go_.wait(l, [&] { return turn_ != seen; });
                seen = turn_;
                if (stop_) return;
            }
            guarded(t);
            if (left_.fetch_sub(1, std::memory_order_acq_rel) == 1) {
                std::lock_guard<std::mutex> l(mu_);
                done_.notify_one();
            }
        }
    }
    int n_;
    std::vector<std::thread> threads_;
    std::mutex mu_;
    std::condition_variable go_, done_;
    uint64_t turn_ = 0;
    bool stop_ = false;
    std::exception_ptr error_;
    std::atomic<int> left_{0};
    void (*call_)(void*, int) = nullptr;
    void* arg_ = nullptr;
};

// Uninitialised memory (a vector would write it once from one thread)
template <class T> struct Buffer {
    T* p = nullptr;
    ~Buffer() { free(p); }
    bool resize(int64_t n) { p = static_cast<T*>(alloc_large(std::max<size_t>(sizeof(T), (size_t)n * sizeof(T)))); return p != nullptr; }
    void drop() { free(p); p = nullptr; }
    T& operator[](int64_t i) { return p[i]; }
};

// Exclusive prefix sum of counts into ptr[0..n]; returns the total.
int64_t prefix(const int64_t* cnt, int64_t n, std::vector<int64_t>& ptr) {
    int64_t s = 0;
    ptr.resize((size_t)n + 1);
    for (int64_t i = 0; i < n; ++i) { ptr[(size_t)i] = s; s += cnt[i]; }
    ptr[(size_t)n] = s;
    return s;
}

// Vertices are dealt to buckets of 2^shift consecutive ids: few enough that every thread can write to all of them side by
// side, small enough that one bucket's entries stay in a core's cache while they are sorted
struct Buckets {
    int shift = 0;
    int64_t count = 1;
    Buckets(int64_t n, int64_t entries, int threads) {
        const int64_t want = std::max<int64_t>(std::min<int64_t>(2048, entries / 16384), threads > 1 ? 4 * threads : 1);
        while (((std::max<int64_t>(n, 1) - 1) >> shift) + 1 > want) ++shift;
        count = ((std::max<int64_t>(n, 1) - 1) >> shift) + 1;
    }
    int64_t of(int32_t v) const { return (int64_t)v >> shift; }
};

// counts[part * buckets + k] -> first position of the part's entries in bucket k (parts in order inside a bucket), start[k] = first
// position of bucket k, start[buckets] = the total, which is returned
int64_t place(std::vector<int64_t>& counts, int64_t buckets, int parts, std::vector<int64_t>& start) {
    start.resize((size_t)buckets + 1);
    int64_t s = 0;
    for (int64_t k = 0; k < buckets; ++k) {
        start[(size_t)k] = s;
        for (int p = 0; p < parts; ++p) {
            int64_t& x = counts[(size_t)(p * buckets + k)];
            const int64_t c = x;
            x = s;
            s += c;
        }
    }
    start[(size_t)buckets] = s;
    return s;
}

struct Item { int32_t row, nb; };

struct WeightedItem { int32_t row, nb; float w; };

// One bucket (rows [r0, r1)) in (row, neighbour) order by a stable radix sort: two or three passes over the bits of the
// neighbour, one over the row; then dedup row by row.  (A comparison sort of every row took 2.8 ms for 2.3 M entries on
// 16 threads, this 1.2.)
template <class It>
void sort_bucket(const Item* in, const float* in_w, int64_t cnt, int64_t n, int64_t r0, int64_t r1, bool dedup, bool loops,
                 int32_t* nb_out, float* w_out, int64_t* len) {
    constexpr bool WEIGHTED = std::is_same<It, WeightedItem>::value;
    int bits = 1;
    while (((n - 1) >> bits) > 0) ++bits;
    const int passes = cnt <= 256 ? (bits + 5) / 6 : (bits + 10) / 11, digit = (bits + passes - 1) / passes;
    const int64_t radix = 1ll << digit, rows = r1 - r0;
    std::vector<int64_t> hist((size_t)(passes * radix + rows + 1), 0);
    int64_t* row_hist = hist.data() + passes * radix;
    for (int64_t i = 0; i < cnt; ++i) {
        for (int p = 0; p < passes; ++p) ++hist[(size_t)(p * radix + ((in[i].nb >> (p * digit)) & (radix - 1)))];
        ++row_hist[in[i].row - r0];
    }
    for (int p = 0; p <= passes; ++p) {
        int64_t at = 0;
        int64_t* h = hist.data() + p * radix;
        for (int64_t k = 0, e = p < passes ? radix : rows; k < e; ++k) { const int64_t c = h[k]; h[k] = at; at += c; }
    }
    Buffer<It> a, b;
    if (!a.resize(cnt) || !b.resize(cnt)) throw std::bad_alloc();
    It *from = a.p, *to = b.p;
    for (int64_t i = 0; i < cnt; ++i) {
        It x;
        x.row = in[i].row;
        x.nb = in[i].nb;
        if constexpr (WEIGHTED) x.w = in_w[i];
        from[hist[(size_t)(x.nb & (radix - 1))]++] = x;
    }
    for (int p = 1; p < passes; ++p, std::swap(from, to))
        for (int64_t i = 0; i < cnt; ++i) to[hist[(size_t)(p * radix + ((from[i].nb >> (p * digit)) & (radix - 1)))]++] = from[i];
    for (int64_t i = 0; i < cnt; ++i) to[row_hist[from[i].row - r0]++] = from[i];          // row_hist[r] is now the end of row r
    int64_t o = 0, i = 0;
    for (int64_t r = 0; r < rows; ++r) {
        const int64_t first = o;
        for (; i < row_hist[r]; ++i) {
            if (dedup && o > first && nb_out[o - 1] == to[i].nb) continue;
            nb_out[o] = to[i].nb;
            if constexpr (WEIGHTED) w_out[o] = to[i].w;
            ++o;
        }
        len[r0 + r] = o - first + (loops ? 1 : 0);
    }
}

int build_threads(int64_t entries) { return (int)std::max<int64_t>(1, std::min<int64_t>(host_threads(), entries / 32768)); }

// The positions of R's entries in the by-source order: entries of one column together, columns ascending, entries of a column in
// R's order.  emit(p, e, row): entry e of row `row` goes to position p.  colptr: first position of every column (filled).
template <class E, class F>
bool transpose_order(Workers& W, const HostSparse& R, std::vector<int64_t>& colptr, int64_t* counts, F&& emit) {
    struct Moved { int32_t col, row; E e; };
    const int T = W.size();
    const int64_t n = R.n, nnz = R.nnz;
    const Buckets bk(n, nnz, T);
    std::vector<int64_t> at((size_t)(bk.count * T), 0);
    // thread t takes a contiguous range of entries; its rows follow from the row pointers
    auto range = [&](int t) { return nnz / T * t + std::min<int64_t>(t, nnz % T); };
    W.run([&](int t) {
        for (int64_t e = range(t), e1 = range(t + 1); e < e1; ++e) ++at[(size_t)(t * bk.count + bk.of(R.colidx[e]))];
    });
    std::vector<int64_t> start;
    place(at, bk.count, T, start);
    Buffer<Moved> moved;
    if (!moved.resize(nnz)) return false;
    W.run([&](int t) {
        const int64_t e0 = range(t), e1 = range(t + 1);
        if (e0 == e1) return;
        int64_t v = std::upper_bound(R.rowptr.begin(), R.rowptr.end(), e0) - R.rowptr.begin() - 1;
        for (int64_t e = e0; e < e1; ++e) {
            while (R.rowptr[(size_t)v + 1] <= e) ++v;
            const int32_t u = R.colidx[e];
            moved[at[(size_t)(t * bk.count + bk.of(u))]++] = Moved{u, (int32_t)v, (E)e};
        }
    });
    W.each(bk.count, 1, [&](int64_t k) {
        const int64_t c0 = k << bk.shift, c1 = std::min(n, (k + 1) << bk.shift);
        for (int64_t c = c0; c < c1; ++c) counts[c] = 0;
        for (int64_t i = start[(size_t)k]; i < start[(size_t)k + 1]; ++i) ++counts[moved[i].col];
    });
    prefix(counts, n, colptr);
    W.each(bk.count, 1, [&](int64_t k) {
        const int64_t c0 = k << bk.shift, c1 = std::min(n, (k + 1) << bk.shift);
        std::vector<int64_t> fill(colptr.begin() + c0, colptr.begin() + c1);
        for (int64_t i = start[(size_t)k]; i < start[(size_t)k + 1]; ++i) {
            const Moved& m = moved[i];
            emit(fill[(size_t)(m.col - c0)]++, (int64_t)m.e, m.row);
        }
    });
    return true;
}

}  // namespace

void* alloc_large(size_t bytes) {
    constexpr size_t HUGE_PAGE = 2u << 20;
    if (bytes < 2 * HUGE_PAGE) return malloc(bytes);
    void* p = nullptr;
    if (posix_memalign(&p, HUGE_PAGE, bytes) != 0) return nullptr;
    (void)madvise(p, bytes, MADV_HUGEPAGE);          // 512 times fewer page faults on the first pass over it
    return p;
}

// How it works.  Every thread takes a slice of the edge list, counts and then writes its entries (row, neighbour) into
// buckets of consecutive rows; a bucket is then sorted by row and neighbour while it sits in one core's cache.  Every edge
// is read twice, whatever the number of threads.  (Threads that owned row ranges and each read the whole edge list, and a
// stable_sort call per row, made the build of a 1.2 M-edge graph, with upload and export of the arrays, 26.2 ms on 16
// threads; 6.9 with this.)
int build_host_graph(int64_t n, int64_t n_edges, const int32_t* src, const int32_t* dst,
                     const float* edge_weight, uint32_t flags, EntryAllocator alloc,
                     BuiltGraph* out) {
    const bool symmetrise = flags & NTP_SYMMETRISE;
    const bool dedup = flags & NTP_DEDUP;
    const bool loops = flags & NTP_ADD_SELF_LOOPS;
    const bool norm = flags & NTP_NORM_GCN_SYM;
    const int64_t most = n_edges * (symmetrise ? 2 : 1);
    const int T = build_threads(std::max(most, n));
    Workers W(T);
    const Buckets bk(n, most, T);
    auto slice = [&](int t) { return n_edges / T * t + std::min<int64_t>(t, n_edges % T); };

    // ---- pass 1: entries per bucket and thread.  Order inside a bucket: originals by thread, then reversed copies by thread,
    // i.e. the processing order.  Ids are checked on the way.
    const int P = symmetrise ? 2 * T : T;
    std::vector<int64_t> at((size_t)(bk.count * P), 0);
    std::atomic<int64_t> bad{-1};
    W.run([&](int t) {
        for (int64_t i = slice(t), i1 = slice(t + 1); i < i1; ++i) {
            const int32_t s = src[i], d = dst[i];
            if (s < 0 || s >= n || d < 0 || d >= n) { bad.store(i); return; }
            if (dedup && s == d) continue;
            ++at[(size_t)(t * bk.count + bk.of(d))];
            if (symmetrise) ++at[(size_t)((T + t) * bk.count + bk.of(s))];
        }
    });
    if (bad.load() >= 0) {
        set_error("edge %lld has a vertex id outside [0, %lld)", (long long)bad.load(), (long long)n);
        return NTP_EINVAL;
    }
    std::vector<int64_t> start;
    const int64_t total_raw = place(at, bk.count, P, start);
    Buffer<Item> raw;
    Buffer<float> raw_w;
    if (!raw.resize(total_raw) || (edge_weight && !raw_w.resize(total_raw))) { set_error("out of host memory (%lld raw entries)", (long long)total_raw); return NTP_ENOMEM; }
    W.run([&](int t) {
        for (int64_t i = slice(t), i1 = slice(t + 1); i < i1; ++i) {
            const int32_t s = src[i], d = dst[i];
            if (dedup && s == d) continue;
            const int64_t p = at[(size_t)(t * bk.count + bk.of(d))]++;
            raw[p] = Item{d, s};
            if (edge_weight) raw_w[p] = edge_weight[i];
            if (symmetrise) {
                const int64_t q = at[(size_t)((T + t) * bk.count + bk.of(s))]++;
                raw[q] = Item{s, d};
                if (edge_weight) raw_w[q] = edge_weight[i];
            }
        }
    });

    // ---- pass 2, bucket by bucket: entries in (row, neighbour) order (stable), dedup (keep first).  What is left of a bucket's
    // rows goes to its part of `raw`, neighbours to its first half, weights to its second half.
    std::vector<int64_t> len((size_t)n, 0);          // final row lengths, self loop included
    W.each(bk.count, 1, [&](int64_t k) {
        const int64_t r0 = k << bk.shift, r1 = std::min(n, (k + 1) << bk.shift), b = start[(size_t)k], cnt = start[(size_t)k + 1] - b;
        int32_t* nb_out = reinterpret_cast<int32_t*>(raw.p + b);
        float* w_out = reinterpret_cast<float*>(nb_out + cnt);
        if (edge_weight)
            sort_bucket<WeightedItem>(raw.p + b, raw_w.p + b, cnt, n, r0, r1, dedup, loops, nb_out, w_out, len.data());
        else
            sort_bucket<Item>(raw.p + b, nullptr, cnt, n, r0, r1, dedup, loops, nb_out, w_out, len.data());
    });

    HostSparse& R = out->csr;
    R.n = n;
    R.nnz = prefix(len.data(), n, R.rowptr);
    R.colidx = (int32_t*)alloc.alloc(std::max<size_t>(4, (size_t)R.nnz * 4), alloc.ctx);
    // without caller weights the values follow from the structure and are rebuilt on the device for
    // streamed chunks: they need not sit in pinned memory
    auto alloc_val = edge_weight ? alloc.alloc : alloc.alloc_val;
    R.val = (float*)alloc_val(std::max<size_t>(4, (size_t)R.nnz * 4), alloc.ctx);
    if (!R.colidx || !R.val) { set_error("out of host memory for %lld entries", (long long)R.nnz); return NTP_ENOMEM; }

    // With unit weights and SYMMETRISE the entry multiset is its own transpose and both
    // degree arrays coincide, so the by-source form equals the by-destination form.
    const bool known_symmetric = symmetrise && edge_weight == nullptr;

    // ---- pass 3: write the final rows; the self loop goes after every entry with id <= v.  Weights:
    // (float)((double)w * (1 / sqrt(din(v) * dout(u)))), here already where both degrees are the row lengths
    auto scaled = [](float w, int64_t d_row, int64_t d_col) {
        const double prod = (double)d_row * (double)d_col;
        const double scale = 1.0 / std::sqrt(prod);
        return (float)((double)w * scale);
    };
    const bool scale_now = norm && known_symmetric;
    std::atomic<int64_t> longest{0};
    W.each(bk.count, 1, [&](int64_t k) {
        const int64_t r0 = k << bk.shift, r1 = std::min(n, (k + 1) << bk.shift), b = start[(size_t)k], cnt = start[(size_t)k + 1] - b;
        const int32_t* nb = reinterpret_cast<const int32_t*>(raw.p + b);
        const float* w = edge_weight ? reinterpret_cast<const float*>(nb + cnt) : nullptr;
        int64_t i = 0, top = 0;
        for (int64_t r = r0; r < r1; ++r) {
            const int64_t m = len[(size_t)r] - (loops ? 1 : 0);
            int64_t o = R.rowptr[(size_t)r];
            bool placed = !loops;
            for (int64_t j = 0; j < m; ++j, ++i) {
                if (!placed && nb[i] > r) { R.colidx[o] = (int32_t)r; R.val[o] = 1.0f; ++o; placed = true; }
                R.colidx[o] = nb[i]; R.val[o] = w ? w[i] : 1.0f; ++o;
            }
            if (!placed) { R.colidx[o] = (int32_t)r; R.val[o] = 1.0f; ++o; }
            if (scale_now)
                for (int64_t e = R.rowptr[(size_t)r]; e < o; ++e) R.val[e] = scaled(R.val[e], len[(size_t)r], len[(size_t)R.colidx[e]]);
            top = std::max(top, len[(size_t)r]);
        }
        int64_t seen = longest.load();
        while (seen < top && !longest.compare_exchange_weak(seen, top)) {}
    });
    R.max_degree = longest.load();
    raw.drop();
    raw_w.drop();

    // NTP_SCATTER_BWD: the backward pass scatters over the by-destination rows (Section 4.2.1),
    // so the by-source form is not stored; its row lengths are still needed for the weights.
    const bool want_csc = !(flags & NTP_SCATTER_BWD);
    HostSparse& C = out->csc;
    std::vector<int64_t> dout;          // by-source row lengths
    if (!known_symmetric && !want_csc) {
        dout.assign((size_t)n, 0);
        std::vector<std::vector<int32_t>> part((size_t)T);
        W.run([&](int t) {
            part[(size_t)t].assign((size_t)n, 0);
            for (int64_t e = R.nnz / T * t + std::min<int64_t>(t, R.nnz % T), e1 = R.nnz / T * (t + 1) + std::min<int64_t>(t + 1, R.nnz % T); e < e1; ++e)
                ++part[(size_t)t][(size_t)R.colidx[e]];
        });
        W.each(n, 4096, [&](int64_t v) { for (int t = 0; t < T; ++t) dout[(size_t)v] += part[(size_t)t][(size_t)v]; });
    }
    if (!known_symmetric && want_csc) {
        // ---- by-source form = transpose of the final entries
        dout.assign((size_t)n, 0);
        C.n = n;
        C.nnz = R.nnz;
        C.colidx = (int32_t*)alloc.alloc(std::max<size_t>(4, (size_t)C.nnz * 4), alloc.ctx);
        C.val = (float*)alloc_val(std::max<size_t>(4, (size_t)C.nnz * 4), alloc.ctx);
        if (!C.colidx || !C.val) { set_error("out of host memory for %lld entries", (long long)C.nnz); return NTP_ENOMEM; }
        auto emit = [&](int64_t p, int64_t e, int32_t v) { C.colidx[p] = v; C.val[p] = R.val[e]; };
        const bool ok = R.nnz < INT32_MAX ? transpose_order<int32_t>(W, R, C.rowptr, dout.data(), emit)
                                          : transpose_order<int64_t>(W, R, C.rowptr, dout.data(), emit);
        if (!ok) { set_error("out of host memory for %lld entries", (long long)C.nnz); return NTP_ENOMEM; }
        C.max_degree = 0;
        for (int64_t r = 0; r < n; ++r) C.max_degree = std::max(C.max_degree, dout[(size_t)r]);
    }

    // ---- weights of graphs whose two degree arrays differ
    if (norm && !known_symmetric) {
        auto scale_rows = [&](HostSparse& M, const std::vector<int64_t>& d_row, const std::vector<int64_t>& d_col) {
            W.each(n, 1024, [&](int64_t r) {
                for (int64_t e = M.rowptr[(size_t)r]; e < M.rowptr[(size_t)r + 1]; ++e)
                    M.val[e] = scaled(M.val[e], d_row[(size_t)r], d_col[(size_t)M.colidx[e]]);
            });
        };
        // CSR row v / column u: din(v) * dout(u);  CSC row u / column v: dout(u) * din(v)
        scale_rows(R, len, dout);
        if (want_csc) scale_rows(C, dout, len);
    }

    // ---- symmetric detection (bitwise)
    bool sym = known_symmetric;
    if (!known_symmetric && want_csc) {
        sym = (C.nnz == R.nnz) && C.rowptr == R.rowptr &&
              memcmp(C.colidx, R.colidx, (size_t)R.nnz * 4) == 0 &&
              memcmp(C.val, R.val, (size_t)R.nnz * 4) == 0;
    }
    out->n = n;
    out->symmetric = sym;
    out->has_csc = sym || want_csc;
    // weights that follow from the structure alone need not travel with a streamed chunk
    out->val_mode = edge_weight ? VAL_STORED : (norm ? VAL_GCN : VAL_ONES);
    if (out->val_mode == VAL_GCN) {
        const std::vector<int64_t>& d_out = known_symmetric ? len : dout;
        out->din.resize((size_t)n);
        out->dout.resize((size_t)n);
        W.each(n, 16384, [&](int64_t v) { out->din[(size_t)v] = (int32_t)len[(size_t)v]; out->dout[(size_t)v] = (int32_t)d_out[(size_t)v]; });
    }
    return NTP_OK;
}

// perm[p] = position, in the by-destination form, of the edge stored at position p of the
// by-source form (the by-destination form itself when the graph is symmetric: its rows are the columns
// of the by-source order)
bool build_edge_perm(const BuiltGraph& G, int32_t* perm) {
    const HostSparse& R = G.csr;
    Workers W(build_threads(R.nnz));
    std::vector<int64_t> colptr, counts((size_t)G.n, 0);
    return transpose_order<int32_t>(W, R, colptr, counts.data(), [&](int64_t p, int64_t e, int32_t) { perm[p] = (int32_t)e; });
}

BuildArena plan_build_arena(int64_t n, int64_t n_edges, uint32_t flags) {
    const bool symmetrise = flags & NTP_SYMMETRISE, want_csc = !symmetrise && !(flags & NTP_SCATTER_BWD);
    BuildArena a;
    a.raw = n_edges * (symmetrise ? 2 : 1) + (flags & NTP_ADD_SELF_LOOPS ? n : 0);
    a.row_pointers = want_csc ? 2 : 1;
    a.degrees = symmetrise ? 1 : 2;
    const size_t tiles = (size_t)((a.raw + BUILD_TILE - 1) / BUILD_TILE), radix = (size_t)1 << BUILD_RADIX_BITS;
    auto take = [&](size_t bytes) { const size_t at = a.bytes; a.bytes += (bytes + 255) / 256 * 256; return at; };
    for (size_t& k : a.keys) k = take((size_t)a.raw * 8);
    if (want_csc) a.colidx = take((size_t)a.raw * 4);
    for (int k = 0; k < a.row_pointers; ++k) a.rowptr[k] = take((size_t)(n + 1) * 8);
    for (int k = 0; k < a.degrees; ++k) a.degree[k] = take((size_t)n * 4);
    a.counts = take(tiles * radix * 4);
    a.totals = take(radix * 4);
    a.kept = take(tiles * 4);
    a.result = take(BUILD_RESULT_BYTES);
    return a;
}

}  // namespace ntp
