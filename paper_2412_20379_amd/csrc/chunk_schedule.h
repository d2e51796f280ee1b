// The order of a pass over chunks of which some are streamed: which stream copies, which stream waits for what, and
// what holds when a pass ends early.  Host logic only; the streams, the copies and the kernels are those of Ops
// (ntp_api.hip: HIP; host_check.cpp: a recorder that checks every access to a staging buffer against the order).
//
// Staging buffers take turns: two that hold a chunk's arrays as the kernels read them, or, where ids travel packed, up to MAX_BUFFERS that hold what
// came over the link (row pointers, lists, packed ids), with one place for the unpacked entries, which belongs to the compute stream alone.
// Whoever writes a buffer waits for its readers (event free_), the readers wait for the
// copy (event ready).  At the end of a pass, completed or not, every buffer that it touched has its free_ event recorded
// behind all copies into it and all kernels on it, and the caller's copy stream stands behind the second one: the next
// pass may come on other streams.
#pragma once

#include <cstdint>
#include <iterator>

namespace ntp {

// How the parts of a streamed chunk travel.
struct CopyPath {
    bool dma;               // entries by DMA on a copy stream; else everything by a kernel on the compute stream (no event)
    bool two_streams;       // the buffers have a copy stream each: the 20-60 us it takes to start a copy pass while the other
                            // one is on the link; else the caller's copy stream takes all copies, one after the other
    bool meta_on_compute;   // row pointers and lists by a kernel on the compute stream, else by one behind the entries
    bool whole = false;     // row pointers, lists and packed ids lie side by side: one copy takes them all
};

// The path for a pass whose streamed chunks have, on average, `bytes` to copy and `entries` entries to aggregate into n_rhs
// right-hand sides of `lines` cache lines a row; largest: bytes of the largest one.  Estimates: 56 GB/s on the link; 10 us a
// launch and 100 G lines/s in the aggregation.
//   Up to 3/4 MB a copy by DMA with its events (50-70 us a chunk whatever its size) costs more than it hides.  us a pass over
//   2.0 M entries, one right-hand side of 32 columns / eight, all on the compute stream against DMA: chunks of 0.1 M entries
//   (0.5 MB) 846 / 1992 against 840 / 2193, 0.2 M 512 / 1099 against 455 / 1141, 0.3 M 408 / 824 against 338 / 822, 0.4 M (1.8 MB)
//   341 / 660 against 266 / 621.
//   Two copies at a time share the link and both arrive late, and the aggregation with them; its time then shows at the ends of
//   a pass.  Hence one at a time where the aggregation is long (0.4 of the copy) and the start of a copy is short against it.
//   us a pass from rest, two streams / one: 4 chunks of 16 M entries, 4 x 32 columns 6539 / 5642, F = 256 9171 / 7835;
//   4 of 4 M F = 256 2063 / 1714; but pass after pass 8 of 2 M F = 128 1499 / 1630.
//   The row pointers and lists (a fifth of the bytes at 15 entries a row) are copied on the compute stream until the
//   aggregation cannot spare the time (0.7 of the copy).  On the compute / copy stream: 4 chunks of 4 M entries F = 32 1268 / 1314,
//   F = 256 1511 / 1438, 8 x 32 columns 1852 / 1762; 11 of 0.4 M F = 32 669 / 682, F = 128 862 / 803, F = 256 1096 / 1016.
//   Packed ids (`packed`) come with their row pointers and lists in one copy, one copy at a time: the buffers that it goes to hold nothing else, so
//   there are more of them than two, and the next copy runs ahead of the kernels.  us for both directions, two images with the row pointers copied by a kernel and two
//   copy streams while the link is the bound / these buffers with two copy streams / with one: 15.8 M entries of 306,128 vertices, chunks of 4 M F = 32
//   1291 / 1300 / 1263, F = 76 1474 / 1625 / 1478, F = 128 1766 / 2360 / 1773; of 1 M F = 32 3062 / 2793 / 1904, F = 76 2460 / 2528 / 2460; of 0.66 M
//   F = 32 3984 / 3701 / 2556; 15 M entries of 1 M vertices in chunks of 2 M F = 32 3181 / 2722 / 2024, F = 128 3582 / 3733 / 3599; 5.1 M of 70,000 in
//   chunks of 1.3 M F = 16 764 / 658 / 508.  By a kernel of 16 blocks on the copy stream instead of by DMA 1555 (chunks of 4 M), 2470 (1 M): what runs
//   beside it waits behind its loads.
inline CopyPath pick_copy_path(double bytes, double largest, double entries, int64_t lines, int n_rhs, bool packed = false) {
    const double copy_us = bytes / 56e3, aggregate_us = n_rhs * (10.0 + entries * (double)lines * 1e-5);
    CopyPath p;
    p.dma = largest > 768 * 1024;
    p.two_streams = p.dma && (aggregate_us < 0.4 * copy_us || copy_us < 200);
    p.meta_on_compute = !p.dma || aggregate_us <= 0.7 * copy_us;
    p.whole = packed;
    if (packed && p.dma) p.two_streams = p.meta_on_compute = false;
    return p;
}

constexpr int MAX_BUFFERS = 4;

template <class Ops> struct StageState {
    typename Ops::Event ready[MAX_BUFFERS] = {}, free_[MAX_BUFFERS] = {}, join[2] = {};
    typename Ops::Stream copy2 = {};        // every other copy's stream where there are two (the others': the caller's)
    bool used[MAX_BUFFERS] = {};            // free_ has been recorded
    int buffers = 2, next = 0, turn = 0;
    int last = -1;                          // the buffer whose kernels used the unpacked entries last
};

// Calls of Ops (0: done, else a status that ends the pass):
//   record(event, stream), wait(stream, event)
//   copy_entries(c, buffer, stream), copy_by_kernel(c, buffer, stream, entries too?)
//   aggregate(c, buffer)   weights rebuilt where they did not travel, and the chunk's kernels; buffer -1: resident
template <class Ops>
class StreamedPass {
public:
    using Stream = typename Ops::Stream;
    StreamedPass(Ops& ops, StageState<Ops>& st, Stream compute, Stream copy, CopyPath path)
        : ops_(ops), st_(st), cs_(compute), xs_(copy), path_(path) {}
    StreamedPass(const StreamedPass&) = delete;
    ~StreamedPass() { if (open_) (void)close(); }      // ended early: nothing more to report

    int begin() {
        open_ = true;
        oldest_ = st_.next;
        if (!path_.two_streams) return 0;
        int rc = ops_.record(st_.join[0], xs_);        // the second copy stream starts where the caller's stands
        if (rc == 0) rc = ops_.wait(st_.copy2, st_.join[0]);
        forked_ = rc == 0;
        return rc;
    }
    // The chunks of a form in order.  Those that lie on the device (is_resident) are run by `resident`.
    // A chunk's copy is enqueued before the kernels of the chunk before it, and the event behind it after them.  HIP deals its streams to four hardware
    // queues; where the copy stream shares the compute stream's (about every fourth stream that a program makes), what waits for a copy holds up everything
    // enqueued behind it, so that copies and kernels alternated.  us a pass, copies enqueued after the kernels / so: 15.8 M entries of 306,128 vertices in
    // chunks of 1 M, F = 32 3300 / 2050 on such a stream (1835 / 1845 on another), 15 M of 539,095 in chunks of 1.7 M, F = 16 3035 / 1770 (1690 / 1690).
    template <class Chunks, class IsResident, class Resident> int run(const Chunks& chunks, IsResident&& is_resident, Resident&& resident) {
        int rc = 0;
        auto ahead = std::begin(chunks);
        const auto end = std::end(chunks);
        bool copied = false;                           // the next streamed chunk's copy is enqueued
        auto copy_next = [&] {
            while (ahead != end && is_resident(*ahead)) ++ahead;
            if (ahead == end) return 0;
            copied = true;
            return copy(*ahead++);
        };
        for (auto c = std::begin(chunks); c != end && rc == 0; ++c) {
            if (is_resident(*c)) { rc = resident(*c); continue; }
            if (!copied) rc = copy_next();
            copied = false;
            const int b = oldest_;
            oldest_ = (b + 1) % st_.buffers;
            if (rc == 0 && path_.dma) rc = ops_.record(st_.ready[b], on_[b]);
            if (rc == 0 && path_.dma && st_.buffers > 1) rc = copy_next();
            if (rc == 0) rc = aggregate(*c, b);
        }
        return rc;
    }
    int end() { return close(); }

private:
    template <class Chunk> int copy(const Chunk& c) {
        const int b = st_.next;
        st_.next = (b + 1) % st_.buffers;
        st_.turn ^= 1;
        const Stream ks = on_[b] = !path_.dma ? cs_ : st_.turn == 0 && path_.two_streams ? st_.copy2 : xs_;
        int rc = 0;
        // the buffer may still be read by the kernels of the chunk that used it last (of an earlier pass: on any stream)
        if (st_.used[b] && !touched_[b]) rc = ops_.wait(cs_, st_.free_[b]);
        if (rc == 0 && st_.used[b] && path_.dma) rc = ops_.wait(ks, st_.free_[b]);
        if (rc != 0) return rc;
        touched_[b] = held_[b] = true;
        if (path_.dma) {
            copying_[b] = true;
            rc = ops_.copy_entries(c, b, ks);
            if (rc == 0 && !path_.meta_on_compute && !path_.whole) rc = ops_.copy_by_kernel(c, b, ks, false);
        }
        return rc;
    }
    template <class Chunk> int aggregate(const Chunk& c, int b) {
        int rc = 0;
        if (path_.whole && !entered_) {       // the unpacked entries: kernels of an earlier pass, on any stream
            if (st_.last >= 0 && st_.used[st_.last]) rc = ops_.wait(cs_, st_.free_[st_.last]);
            entered_ = rc == 0;
        }
        if (rc == 0 && path_.meta_on_compute && !(path_.whole && path_.dma)) rc = ops_.copy_by_kernel(c, b, cs_, !path_.dma);
        if (rc == 0 && path_.dma) {
            rc = ops_.wait(cs_, st_.ready[b]);
            if (rc == 0) copying_[b] = false;
        }
        if (rc == 0) {
            st_.last = b;
            rc = ops_.aggregate(c, b);
        }
        if (rc != 0 || !path_.dma) return rc;
        return release(b);
    }
    int release(int b) {
        const int rc = ops_.record(st_.free_[b], cs_);
        if (rc == 0) { st_.used[b] = true; held_[b] = false; }
        return rc;
    }
    // goes on after a failure: what can be put in order is
    int close() {
        open_ = false;
        int rc = 0;
        auto also = [&](int r) { if (rc == 0) rc = r; return r == 0; };
        for (int b = 0; b < MAX_BUFFERS; ++b) {
            if (copying_[b] && also(ops_.record(st_.ready[b], on_[b]))) also(ops_.wait(cs_, st_.ready[b]));
            copying_[b] = false;
            if (held_[b]) also(release(b));
        }
        // whoever waits for the caller's copy stream waits for all copies
        if (forked_ && also(ops_.record(st_.join[1], st_.copy2))) also(ops_.wait(xs_, st_.join[1]));
        forked_ = false;
        return rc;
    }

    Ops& ops_;
    StageState<Ops>& st_;
    const Stream cs_, xs_;
    const CopyPath path_;
    bool open_ = false, forked_ = false, entered_ = false;
    int oldest_ = 0;                        // the buffer whose kernels come next
    Stream on_[MAX_BUFFERS] = {};           // of the buffer's copy
    bool touched_[MAX_BUFFERS] = {};        // the compute stream has waited for the buffer's earlier readers
    bool copying_[MAX_BUFFERS] = {};        // a copy is enqueued that the compute stream does not wait for yet
    bool held_[MAX_BUFFERS] = {};           // used since free_ was recorded last
};

}  // namespace ntp
