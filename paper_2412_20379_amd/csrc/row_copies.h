// The making of the second copies of a resident chunk (see RowCopies).  Host logic only; the memory and the kernels are those of
// Ops (ntp_api.hip: HIP; host_check.cpp: host memory, with a failure at every step).
#pragma once

#include <new>

#include "ntp_internal.h"

namespace ntp {

// The copies are an addition: where they do not fit, on the device or in host memory, the chunk goes on with the form's own
// arrays.  Only a call of the runtime that fails otherwise ends the build.
// Calls of Ops:
//   alloc(bytes)      device memory, nullptr: not to be had
//   release(p)
//   upload(p, src, bytes), fill_slices(chunk, layout, p, bin), fill_packed(chunk, layout, p)      0: done, else a status
template <class Ops> int make_row_copies(Ops& ops, const HostSparse& m, Chunk& c) {
    RowCopies layout;
    std::vector<char> lists;
    try {
        plan_row_copies(m, c, &layout, &lists);
    } catch (const std::bad_alloc&) {
        return 0;
    }
    if (layout.bytes == 0) return 0;
    char* p = ops.alloc(layout.bytes);
    if (!p) return 0;
    int rc = ops.upload(p + layout.off_lists, lists.data(), lists.size());
    if (layout.slices)
        for (int b = 0; b < SLICE_BINS && rc == 0; ++b) rc = ops.fill_slices(c, layout, p, b);
    if (layout.packed_rows > 0 && rc == 0) rc = ops.fill_packed(c, layout, p);
    if (rc != 0) {
        ops.release(p);
        return rc;
    }
    c.d_copies = p;
    c.copies = layout;
    return 0;
}

}  // namespace ntp
