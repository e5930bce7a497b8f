// Descriptors and launchers of the persistent tile kernel shared by the batch
// and serving runtimes (internal to librc).
#pragma once

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

#include "rc.h"
#include "runtime.h"

namespace rc {

constexpr int kBatchThreads = 1024;
// Threads of a workgroup that stream the image; all build the LUT strip.
constexpr int kBatchStream = 256;
// Lines per register set.
constexpr int kBatchUnroll = 4;
constexpr size_t kBatchLds = 80 * 1024;
// Resident workgroups per CU (1024 threads of up to 128 registers).
constexpr int kBatchPerCu = 1;
// Tile queues of the persistent kernel: one per XCD (workgroups are dispatched
// to the XCDs round-robin, so workgroup i starts on queue i % kBatchQueues).
constexpr int kBatchQueues = 8;
// Device counters of one launch: a head per queue, then the number of
// workgroups that have finished.
constexpr int kBatchCounters = kBatchQueues + 1;

// Per-request descriptor, resident in device memory.
struct BatchReq {
    const double* coeffs;
    const uint16_t* dn;
    uint16_t* lut;
    uint16_t* out;
    int64_t lines;
    int32_t detectors;
    int32_t bands;
    int32_t levels;
    int32_t log_strip;
    int32_t vec;
    int32_t mode;     // kRaw / kGlobal / kPacked / kDense
    int32_t lut_vec;  // LUT rows allow 16-byte loads/stores
    int32_t fused;    // tiles build their LUT strip in LDS (all modes but kGlobal)
    int32_t pad;
};

// First detector of strip s, and the width of the strip that starts at d0.
// Where the rest of a row is less than the 8 detectors a lane takes, the last
// strip takes what it lacks from the one before it, so that strips stay apart
// (a request may be corrected in place); strips of 8 overlap instead.
constexpr int32_t strip_start(const BatchReq& q, int32_t s) {
    const int32_t d0 = s << q.log_strip;
    return q.vec == 8 && q.detectors - d0 < 8 ? q.detectors - 8 : d0;
}
constexpr int32_t strip_width(const BatchReq& q, int32_t d0) {
    const int32_t W = 1 << q.log_strip;
    const int32_t after = q.detectors - d0 - W;
    if (q.vec == 8 && W > 8 && after > 0 && after < 8) return W - (8 - after);
    return after < 0 ? W + after : W;
}

struct BatchTile {
    int32_t req;
    int32_t band;
    int32_t d0;
    int32_t pad;
    int64_t n0;
    int64_t n1;
};

// Queue q holds tiles [bound[q], bound[q + 1]); bound is non-decreasing from
// 0 to the tile count. A single queue is bound = {0, n, n, ..., n}.
struct BatchQueues {
    int32_t bound[kBatchQueues + 1];
};

// Persistent correction kernel: each of the `grid` workgroups pops tiles
// from its own queue, then from the others until every queue is empty.
// `counters` holds kBatchCounters zeros before the first launch; the kernel
// rearms them itself.
hipError_t launch_batch_apply(const BatchReq* reqs, const BatchTile* tiles,
                              const BatchQueues& queues, unsigned int* counters, int grid,
                              size_t lds, hipStream_t stream);

// Queues holding tiles [0, n) in one queue.
BatchQueues single_queue(int32_t n);

// Sets the persistent kernel's dynamic LDS limit on the current device.
hipError_t prepare_batch_kernel(size_t lds);

// Fills q's strip shape and mode from a plan, fitted to the persistent
// kernel's workgroup size and LDS budget; 8 pixels per lane whatever the rows'
// alignment, except for fewer than 8 detectors, and in place where strips of 8
// would have to overlap.
void fit_request_plan(const rc_plan& plan, int levels, size_t lds_cap, BatchReq* q);

}  // namespace rc
