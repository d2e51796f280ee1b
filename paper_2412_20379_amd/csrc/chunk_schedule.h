// The order of a pass over chunks of which some are streamed: which stream copies, which stream waits for what, and
// what holds when a pass ends early.  Host logic only; the streams, the copies and the kernels are those of Ops
// (ntp_api.hip: HIP; host_check.cpp: a recorder that checks every access to a staging buffer against the order).
//
// Two staging buffers alternate.  Whoever writes a buffer waits for its readers (event free_), the readers wait for the
// copy (event ready).  At the end of a pass, completed or not, every buffer that it touched has its free_ event recorded
// behind all copies into it and all kernels on it, and the caller's copy stream stands behind the second one: the next
// pass may come on other streams.
#pragma once

#include <cstdint>

namespace ntp {

// How the parts of a streamed chunk travel.
struct CopyPath {
    bool dma;               // entries by DMA on a copy stream; else everything by a kernel on the compute stream (no event)
    bool two_streams;       // the buffers have a copy stream each: the 20-60 us it takes to start a copy pass while the other
                            // one is on the link; else the caller's copy stream takes all copies, one after the other
    bool meta_on_compute;   // row pointers and lists by a kernel on the compute stream, else by one behind the entries
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
//   Packed ids (`packed`) are a half to seven eighths of the bytes, and kernels that unpack them and rebuild the weights stand before the
//   aggregation: by these bounds two copies at a time and row pointers on the compute stream would hold up a pass that the aggregation
//   already bounds.  From three lines a row on: one copy at a time, the row pointers behind it.  us for both directions, ids as they are /
//   packed by these bounds / packed and so: 4 chunks of 4 M entries of 306,128 vertices F = 76 2840 / 2819 / 2448, F = 128 3019 / 3049 / 2852,
//   of 200,000 F = 160 3175 / 3460 / 3198; 16 of 1 M of 1 M vertices F = 76 4045 / 4004 / 3504; 23 of 0.7 M of 306,128 F = 128 4373 / 4498 /
//   4372.  Fewer lines stay with the bounds: 4 of 4 M of 306,128 F = 32 2769 / 1789 / 1948, of 200,000 F = 64 2869 / 1815 / 1940.
inline CopyPath pick_copy_path(double bytes, double largest, double entries, int64_t lines, int n_rhs, bool packed = false) {
    const double copy_us = bytes / 56e3, aggregate_us = n_rhs * (10.0 + entries * (double)lines * 1e-5);
    CopyPath p;
    p.dma = largest > 768 * 1024;
    p.two_streams = p.dma && (aggregate_us < 0.4 * copy_us || copy_us < 200);
    p.meta_on_compute = !p.dma || aggregate_us <= 0.7 * copy_us;
    if (packed && p.dma && n_rhs * lines > 2) p.two_streams = p.meta_on_compute = false;
    return p;
}

template <class Ops> struct StageState {
    typename Ops::Event ready[2] = {}, free_[2] = {}, join[2] = {};
    typename Ops::Stream copy2 = {};        // buffer 1's copy stream where there are two (buffer 0's is the caller's)
    bool used[2] = {false, false};          // free_ has been recorded
    int next = 0;
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
        if (!path_.two_streams) return 0;
        int rc = ops_.record(st_.join[0], xs_);        // the second copy stream starts where the caller's stands
        if (rc == 0) rc = ops_.wait(st_.copy2, st_.join[0]);
        forked_ = rc == 0;
        return rc;
    }
    template <class Chunk> int streamed(const Chunk& c) {
        const int b = st_.next;
        st_.next ^= 1;
        const Stream ks = path_.dma ? copy_stream(b) : cs_;
        int rc = 0;
        // the buffer may still be read by the kernels of the chunk that used it last (of an earlier pass: on any stream)
        if (st_.used[b] && !touched_[b]) rc = ops_.wait(cs_, st_.free_[b]);
        if (rc == 0 && st_.used[b] && path_.dma) rc = ops_.wait(ks, st_.free_[b]);
        if (rc != 0) return rc;
        touched_[b] = held_[b] = true;
        if (path_.dma) {
            copying_[b] = true;
            rc = ops_.copy_entries(c, b, ks);
            if (rc == 0 && !path_.meta_on_compute) rc = ops_.copy_by_kernel(c, b, ks, false);
            if (rc == 0) rc = ops_.record(st_.ready[b], ks);
        }
        if (rc == 0 && path_.meta_on_compute) rc = ops_.copy_by_kernel(c, b, cs_, !path_.dma);
        if (rc == 0 && path_.dma) {
            rc = ops_.wait(cs_, st_.ready[b]);
            if (rc == 0) copying_[b] = false;
        }
        if (rc == 0) rc = ops_.aggregate(c, b);
        if (rc != 0 || !path_.dma) return rc;
        return release(b);
    }
    int end() { return close(); }

private:
    Stream copy_stream(int b) const { return b == 1 && path_.two_streams ? st_.copy2 : xs_; }
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
        for (int b = 0; b < 2; ++b) {
            if (copying_[b] && also(ops_.record(st_.ready[b], copy_stream(b)))) also(ops_.wait(cs_, st_.ready[b]));
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
    bool open_ = false, forked_ = false;
    bool touched_[2] = {false, false};      // the compute stream has waited for the buffer's earlier readers
    bool copying_[2] = {false, false};      // a copy is enqueued that the compute stream does not wait for yet
    bool held_[2] = {false, false};         // used since free_ was recorded last
};

}  // namespace ntp
