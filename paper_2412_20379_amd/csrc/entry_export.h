// Reading a form's entries back from the images of its chunks (a graph built on the device has no others).  Host logic only; the device, the
// stream and the copies are those of Ops (ntp_api.hip: HIP; host_check.cpp: a recorder with a failure at every call).
#pragma once

#include "ntp_internal.h"

namespace ntp {

// The caller may have another device current, or a stream under capture: the copies go to the graph's device, and what the caller's thread had is
// there again afterwards, in any case.
// Calls of Ops (0: done, else a status):
//   exchange_capture_mode()                 first to one that permits copies, then back
//   current_device(int*), set_device(int)
//   begin()                                 a stream of the current device for the copies
//   copy(dst, src, bytes), finish()         enqueued; waited for
template <class Ops> int read_entries(Ops& ops, int device, const std::vector<Chunk>& chunks, int32_t* colidx, float* val) {
    int rc = ops.exchange_capture_mode();
    if (rc != 0) return rc;
    auto also = [&](int r) { if (rc == 0) rc = r; return r == 0; };
    int before = device;
    bool away = false;
    if (also(ops.current_device(&before)) && before != device) away = also(ops.set_device(device));
    if (rc == 0 && also(ops.begin())) {
        for (const Chunk& c : chunks) {
            const size_t bytes = (size_t)(c.e_end - c.e_begin) * 4;
            if (bytes && colidx && rc == 0) also(ops.copy(colidx + c.e_begin, c.d_image + c.img_off_colidx, bytes));
            if (bytes && val && rc == 0) also(ops.copy(val + c.e_begin, c.d_image + c.img_off_val, bytes));
        }
        also(ops.finish());
    }
    if (away) also(ops.set_device(before));
    also(ops.exchange_capture_mode());
    return rc;
}

}  // namespace ntp
