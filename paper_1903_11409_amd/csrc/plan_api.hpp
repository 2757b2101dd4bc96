// What the Python binding and the tests ask a plan beside the C ABI: creation from arrays in host memory,
// covered rows, the kernel a product takes.
#pragma once

#include <cstddef>
#include <cstdint>

#include "../../include/bspmm.h"

namespace bspmm {

// `bytes` (a multiple of 256) that write(from, to) puts in front of the plan's tables.
struct HostFront {
    size_t bytes;
    void (*write)(const void* from, char* to);
    const void* from;
};

// bspmm_create for a workspace at `workspace` whose front memory [workspace - front.bytes, workspace)
// is the device home of the arrays `front` writes; `b` names them by their device addresses.  The
// host arrays are read during the call.  ESTATE when they cannot be staged (too large, or the stream
// is being captured): the caller then copies them itself and calls bspmm_create.
int create_from_host(bspmm_plan** plan, const bspmm_batch* b, int32_t F, const bspmm_options* options,
                     void* workspace, size_t workspace_bytes, const HostFront& front, void* stream);

// Returns when the plan's tables are on the device; EHIP when they will not get there.
int settle_upload(bspmm_plan* plan);

// Work enqueued on `stream` from now on runs after what `earlier` holds.  Recording streams are left alone:
// the order inside a graph is its maker's.
int run_after(void* stream, void* earlier);

// Returns when everything that `stream` holds has run (a recording stream: at once); EHIP when it failed.
int run_out(void* stream);

// Rows from the first on, without a gap, that belong to an operation's output: of C, or of G with
// `transposed`.
int64_t covered_rows(bspmm_plan* plan, bool transposed);

// Whether a product with these leading dimensions, on operands aligned to 16 bytes, runs in the lean kernel.
bool takes_lean_kernel(const bspmm_plan* plan, bool transposed, int64_t ld_in, int64_t ld_out);

}  // namespace bspmm
