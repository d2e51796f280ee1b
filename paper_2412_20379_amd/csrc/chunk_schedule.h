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
//   COPY_ON_COMPUTE   everything by a kernel on the compute stream: no event, no second stream
//   COPY_META_ON_COMPUTE  entries by DMA on two copy streams in turn (one per buffer; the 20-30 us it takes to start a copy pass
//                     while the other one is on the link), row pointers and lists by a kernel on the compute stream (four
//                     chunks of 4 M entries: 1.45 -> 1.32 ms a pass, the link alone 1.15)
//   COPY_ON_COPY      the same with the row pointers and lists behind the entries on the copy stream
enum CopyPath { COPY_ON_COMPUTE, COPY_META_ON_COMPUTE, COPY_ON_COPY };

// Up to 2 MB (36 us on the link) a chunk with DMA copies, events and a second stream costs 50-70 us whatever its size.
inline CopyPath pick_copy_path(int64_t largest) { return largest <= (2 << 20) ? COPY_ON_COMPUTE : COPY_META_ON_COMPUTE; }

template <class Ops> struct StageState {
    typename Ops::Event ready[2] = {}, free_[2] = {}, join[2] = {};
    typename Ops::Stream copy2 = {};        // buffer 1's copy stream (buffer 0's is the caller's)
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
        if (path_ == COPY_ON_COMPUTE) return 0;
        int rc = ops_.record(st_.join[0], xs_);        // the second copy stream starts where the caller's stands
        if (rc == 0) rc = ops_.wait(st_.copy2, st_.join[0]);
        forked_ = rc == 0;
        return rc;
    }
    template <class Chunk> int streamed(const Chunk& c) {
        const int b = st_.next;
        st_.next ^= 1;
        const Stream ks = path_ == COPY_ON_COMPUTE ? cs_ : copy_stream(b);
        int rc = 0;
        // the buffer may still be read by the kernels of the chunk that used it last (of an earlier pass: on any stream)
        if (st_.used[b] && !touched_[b]) rc = ops_.wait(cs_, st_.free_[b]);
        if (rc == 0 && st_.used[b] && path_ != COPY_ON_COMPUTE) rc = ops_.wait(ks, st_.free_[b]);
        if (rc != 0) return rc;
        touched_[b] = held_[b] = true;
        if (path_ != COPY_ON_COMPUTE) {
            copying_[b] = true;
            rc = ops_.copy_entries(c, b, ks);
            if (rc == 0 && path_ == COPY_ON_COPY) rc = ops_.copy_by_kernel(c, b, ks, false);
            if (rc == 0) rc = ops_.record(st_.ready[b], ks);
        }
        if (rc == 0 && path_ != COPY_ON_COPY) rc = ops_.copy_by_kernel(c, b, cs_, path_ == COPY_ON_COMPUTE);
        if (rc == 0 && path_ != COPY_ON_COMPUTE) {
            rc = ops_.wait(cs_, st_.ready[b]);
            if (rc == 0) copying_[b] = false;
        }
        if (rc == 0) rc = ops_.aggregate(c, b);
        if (rc != 0 || path_ == COPY_ON_COMPUTE) return rc;
        return release(b);
    }
    int end() { return close(); }

private:
    Stream copy_stream(int b) const { return b == 0 ? xs_ : st_.copy2; }
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
