// Batched execution of many uneven correction requests (§I's LUT generation
// and image correction, run for a whole queue of client scenes at once).
//
// Up to two kernels per run, captured once into a hipGraph and replayed:
//  1. k_lut_build_batch: the LUT entries of the requests that are corrected
//     from the global LUT (the L2 path, for level counts whose strips do not
//     fit LDS); a thread finds its request by binary search over the prefix
//     of work items.
//  2. k_apply_batch: a persistent kernel (one workgroup per resident slot)
//     whose workgroups pop tiles (request, band, strip, lines) from atomic
//     queue heads, one queue per XCD: a workgroup drains its own XCD's queue,
//     then helps with the others. For every other request a tile is fused: it
//     evaluates its strip's LUT rows from the coefficients straight into LDS
//     (the first line chunk of a strip also writes them to the request's LUT),
//     then corrects its lines, so the LUT is never read back from memory.
//     The strips of one request line chunk stay together on one queue,
//     groups are dealt longest first, so the tail of the batch is made of
//     short tiles. The last workgroup to finish resets the counters, so a
//     replay needs no memset node.
// Strip width and LDS mode per request come from its batch entry of the plan
// cache or from batch_plan, fitted to the kernel's workgroup size and LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <new>
#include <type_traits>
#include <vector>

#include "batch.h"
#include "device_ops.h"
#include "kernels.h"
#include "rc.h"
#include "runtime.h"

namespace rc {

__global__ __launch_bounds__(256) void k_lut_build_batch(const BatchReq* __restrict__ reqs,
                                                         const int64_t* __restrict__ prefix,
                                                         int32_t nreq, int64_t total) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * blockDim.x) {
        // Request r owns work items [prefix[r], prefix[r + 1]).
        int lo = 0, hi = nreq - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (prefix[mid] <= t) lo = mid;
            else hi = mid - 1;
        }
        const BatchReq& q = reqs[lo];
        const int L = q.levels;
        const int chunks = (L + 7) >> 3;
        const int64_t local = t - prefix[lo];
        const int64_t row = local / chunks;
        const int c = (int)(local - row * chunks);
        const double* a = q.coeffs + row * 4;
        const double a0 = a[0], a1 = a[1], a2 = a[2], a3 = a[3];
        const int v0 = c * 8;
        double x[8];
        levels8(v0, x);
        store_lut8(q.lut + row * (int64_t)L + v0,
                   lut_eight(a0, a1, a2, a3, x, (uint32_t)(L - 1) * 0x10001u), L - v0,
                   q.lut_vec != 0, false);
    }
}

template <int VEC>
__device__ __forceinline__ void batch_tile_vec(const BatchReq& q, const BatchTile& tl,
                                               void* smem) {
    const int weff = strip_width(q, tl.d0);
    if (q.fused) {
        const bool write_lut = tl.n0 == 0;
        auto run = [&](auto mode) {
            fused_tile<VEC, kBatchUnroll, decltype(mode)::value>(
                q.coeffs, q.dn, q.lut, q.out, q.lines, q.detectors, q.levels, q.log_strip, tl.band,
                tl.d0, weff, tl.n0, tl.n1, write_lut, smem, q.lut_vec != 0, kBatchStream);
        };
        if (q.mode == kPacked) run(std::integral_constant<int, kPacked>{});
        else if (q.mode == kDense) run(std::integral_constant<int, kDense>{});
        else run(std::integral_constant<int, kRaw>{});
    } else {
        apply_tile<VEC, kBatchUnroll, 0, kGlobal>(q.dn, q.lut, q.out, q.lines, q.detectors,
                                                  q.levels, q.log_strip, tl.band, tl.d0, weff,
                                                  tl.n0, tl.n1, smem, q.lut_vec != 0, false);
    }
}

// counters[q]: next tile of queue q; counters[kBatchQueues]: workgroups finished.
// One workgroup of kBatchThreads runs per CU, 4 waves per SIMD: all of it
// evaluates a strip, then 256 threads stream (16 bytes x 4 lines per lane and
// register set). Evaluating a strip is bound by instruction issue and takes a
// CU about as long as streaming 4 bytes per entry (detector_cost), so a batch
// of few tiles lasts as long as one tile's evaluation: as many waves as fit, and
// strips no wider than streaming needs. In us, against two workgroups of 512
// threads per CU and dense strips of 128 detectors at 4096 levels: one request
// of 2 x 1013 x 1492 71 (172), one of 1 x 7009 x 2155 100 (219), 4 of together
// 385 Mpix 557 (690), the 16 of the performance cases 1631 (1750). With 512
// threads streaming: 1 % more on average, up to 10 %.
__global__ __launch_bounds__(kBatchThreads)
void k_apply_batch(const BatchReq* __restrict__ reqs, const BatchTile* __restrict__ tiles,
                   BatchQueues queues, unsigned int* counters) {
    extern __shared__ __align__(16) unsigned char smem[];
    // The popped tile index is broadcast through the first word of the tile
    // LDS, which is dead between tiles (every tile ends with a barrier): no
    // static LDS, so two 80 KiB workgroups fit one CU.
    int* s_tile = (int*)smem;
    // The workgroup's own XCD queue first (neighbouring strips of one request
    // line chunk share that XCD's L2), then whatever the other queues still hold.
    const int home = (int)(blockIdx.x % kBatchQueues);
    for (int k = 0; k < kBatchQueues; ++k) {
        const int qi = (home + k) % kBatchQueues;
        const int lo = queues.bound[qi];
        const int n = queues.bound[qi + 1] - lo;
        for (;;) {
            if (threadIdx.x == 0) *s_tile = (int)atomicAdd(&counters[qi], 1u);
            __syncthreads();
            // Uniform across the workgroup: descriptor loads become scalar loads.
            const int t = __builtin_amdgcn_readfirstlane(*s_tile);
            __syncthreads();
            if (t >= n) break;
            const BatchTile tl = tiles[lo + t];
            const BatchReq q = reqs[tl.req];
            if (q.vec == 8) batch_tile_vec<8>(q, tl, smem);
            else batch_tile_vec<1>(q, tl, smem);
        }
    }
    if (threadIdx.x == 0) {
        const unsigned int done = atomicAdd(&counters[kBatchQueues], 1u);
        if (done == gridDim.x - 1) {
            // Every workgroup has made its last pop: rearm for the next run.
            for (int c = 0; c < kBatchCounters; ++c) atomicExch(&counters[c], 0u);
        }
    }
}

hipError_t launch_batch_apply(const BatchReq* reqs, const BatchTile* tiles,
                              const BatchQueues& queues, unsigned int* counters, int grid,
                              size_t lds, hipStream_t stream) {
    hipLaunchKernelGGL(k_apply_batch, dim3((unsigned)grid), dim3(kBatchThreads), lds, stream, reqs,
                       tiles, queues, counters);
    return hipGetLastError();
}

BatchQueues single_queue(int32_t n) {
    BatchQueues q;
    q.bound[0] = 0;
    for (int i = 1; i <= kBatchQueues; ++i) q.bound[i] = n;
    return q;
}

hipError_t prepare_batch_kernel(size_t lds) {
    // The dense tiles address LDS from byte 0: no static LDS may precede the
    // dynamic buffer.
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, (const void*)k_apply_batch);
    if (e != hipSuccess) return e;
    if (attr.sharedSizeBytes != 0) return hipErrorInvalidImage;
    return hipFuncSetAttribute((const void*)k_apply_batch,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

// Tile shape of a request without a batch entry: the plain path's tuned plan
// if the cache has one, else pow2_plan's (packed strips of 64 detectors at 4096
// levels). Dense strips hold twice the detectors in the same LDS, which makes
// half the tiles, each of twice the evaluation: 51 batches of 1 to 16 requests
// took 1.21 times as long with them on average, between 0.93 and 2.2.
static void batch_plan(int64_t lines, int32_t detectors, int32_t bands, int32_t levels, int vmax,
                       const DeviceInfo& di, rc_plan* plan) {
    if (!tuned_plan(lines, detectors, bands, levels, vmax, di, plan))
        pow2_plan(lines, detectors, bands, levels, vmax, di, plan);
}

void fit_request_plan(const rc_plan& plan_in, int levels, size_t lds_cap, BatchReq* q) {
    rc_plan p = plan_in;
    if (p.path == RC_PATH_DENSE && levels > kDenseMaxLevels) p.path = RC_PATH_PACKED;
    while (p.path != RC_PATH_L2 && plan_lds_bytes(p.path, p.strip, levels) > lds_cap && p.strip > 1)
        p.strip >>= 1;
    if (p.path != RC_PATH_L2 && plan_lds_bytes(p.path, p.strip, levels) > lds_cap)
        p.path = RC_PATH_L2;
    // In place, a line's overlapping lanes share a wave (strips of at most 512
    // detectors), and strips may not overlap (strip_width).
    const bool in_place = q->dn == q->out;
    if (in_place) p.strip = std::min(p.strip, 512);
    const int rest = q->detectors % p.strip;
    p.vec = p.strip >= 8 && q->detectors >= 8 && !(in_place && p.strip == 8 && rest > 0) ? 8 : 1;
    while (p.strip / p.vec > kBatchStream) p.strip >>= 1;
    int lw = 0;
    while ((1 << (lw + 1)) <= p.strip) ++lw;
    q->log_strip = lw;
    q->vec = p.vec;
    q->mode = p.path == RC_PATH_LDS      ? kRaw
              : p.path == RC_PATH_PACKED ? kPacked
              : p.path == RC_PATH_DENSE  ? kDense
                                         : kGlobal;
    q->fused = q->mode != kGlobal ? 1 : 0;
}

}  // namespace rc

using namespace rc;

struct rc_batch {
    int device = 0;
    int32_t nreq = 0;
    int32_t ntiles = 0;
    int64_t build_items = 0;
    int slots = 0;
    int cus = 0;
    size_t lds = 0;
    BatchReq* d_reqs = nullptr;
    BatchTile* d_tiles = nullptr;
    int64_t* d_prefix = nullptr;
    unsigned int* d_counters = nullptr;
    BatchQueues queues{};
    hipStream_t cap = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    bool use_graph = true;
    rc_batch_stats stats{};
};

namespace {

void release(rc_batch* b) {
    if (!b) return;
    // Teardown: failures here have no one left to report to.
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    if (b->cap) (void)hipStreamDestroy(b->cap);
    if (b->d_reqs) (void)hipFree(b->d_reqs);
    if (b->d_tiles) (void)hipFree(b->d_tiles);
    if (b->d_prefix) (void)hipFree(b->d_prefix);
    if (b->d_counters) (void)hipFree(b->d_counters);
    delete b;
}

enum Role { kCoeffs = 0, kLut = 1, kDn = 2, kOut = 3 };

struct Range {
    uintptr_t lo, hi;
    int req;
    int role;
    bool written() const { return role == kLut || role == kOut; }
};

// A buffer written by one request may not overlap any other buffer, read or
// written, of any request. The one exception is a request corrected in
// place: its out may be exactly its own dn. (Within a request, fused tiles
// read the coefficients while other tiles already write the image, so an
// out that overlaps its own coefficients would race.)
bool hazards(const std::vector<Range>& rs) {
    for (size_t a = 0; a < rs.size(); ++a) {
        if (!rs[a].written()) continue;
        for (size_t b = 0; b < rs.size(); ++b) {
            if (a == b) continue;
            if (rs[b].req == rs[a].req && rs[a].role == kOut && rs[b].role == kDn &&
                rs[a].lo == rs[b].lo && rs[a].hi == rs[b].hi)
                continue;  // in place
            if (rs[a].lo < rs[b].hi && rs[b].lo < rs[a].hi) return true;
        }
    }
    return false;
}

// Validates every request and the hazards between them (host only).
rc_status validate_requests(const rc_request* reqs, int32_t n) {
    std::vector<Range> ranges;
    for (int32_t i = 0; i < n; ++i) {
        const rc_request& r = reqs[i];
        if (r.lines < 0 || r.detectors < 0 || r.bands < 0 || r.reserved != 0) return RC_EINVAL;
        if (r.levels < RC_LEVELS_MIN || r.levels > RC_LEVELS_MAX) return RC_EINVAL;
        int64_t px = 0, rows = 0, lut_n = 0;
        if (!mul_ok(r.lines, r.detectors, &px) || !mul_ok(px, r.bands, &px) ||
            !mul_ok((int64_t)r.bands, r.detectors, &rows) || !mul_ok(rows, r.levels, &lut_n) ||
            px > INT64_MAX / 2 || lut_n > INT64_MAX / 2)
            return RC_EINVAL;
        if (rows > 0) {
            if (!r.coeffs || !r.lut || ((uintptr_t)r.coeffs & 7u) || ((uintptr_t)r.lut & 1u))
                return RC_EINVAL;
            ranges.push_back({(uintptr_t)r.lut, (uintptr_t)r.lut + (uintptr_t)lut_n * 2, i, kLut});
            ranges.push_back({(uintptr_t)r.coeffs, (uintptr_t)r.coeffs + (uintptr_t)rows * 32, i,
                              kCoeffs});
        }
        if (px > 0) {
            if (!r.dn || !r.out || (((uintptr_t)r.dn | (uintptr_t)r.out) & 1u)) return RC_EINVAL;
            ranges.push_back({(uintptr_t)r.out, (uintptr_t)r.out + (uintptr_t)px * 2, i, kOut});
            ranges.push_back({(uintptr_t)r.dn, (uintptr_t)r.dn + (uintptr_t)px * 2, i, kDn});
        }
    }
    return hazards(ranges) ? RC_EINVAL : RC_OK;
}

hipError_t enqueue(const rc_batch* b, hipStream_t s) {
    if (b->build_items > 0) {
        int64_t blocks = (b->build_items + 255) / 256;
        if (blocks > ((int64_t)1 << 20)) blocks = (int64_t)1 << 20;
        hipLaunchKernelGGL(k_lut_build_batch, dim3((unsigned)blocks), dim3(256), 0, s, b->d_reqs,
                           b->d_prefix, b->nreq, b->build_items);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (b->ntiles > 0) {
        return launch_batch_apply(b->d_reqs, b->d_tiles, b->queues, b->d_counters, b->slots,
                                  b->lds, s);
    }
    return hipSuccess;
}

}  // namespace

namespace {

// Cost of one detector's part of a tile, in image bytes: reading and writing
// its lines, and evaluating its LUT row in a fused tile, which takes a
// workgroup as long as 4 bytes per entry (1.1 entries and 1.1 pixels per ns
// on the whole GPU), or reading it.
int64_t detector_cost(const BatchReq& q, int64_t lines) {
    return lines * 4 + (int64_t)q.levels * (q.fused ? 4 : 2);
}

// Line chunks of every request. A tile evaluates its strip whatever lines it
// has, so fewer chunks are less work, but the last tiles to finish leave the
// other workgroups idle: the batch takes the longest tile's time if every tile
// has a workgroup, else about the workgroups' share of the work plus 0.6 of
// the longest tile (fitted to a simulation of the queues with 4 to 16 requests
// of 512 to 8192 lines and detectors). Tries bounds on the longest tile and
// takes the best: 36 batches of 1 to 16 requests took 1.12 times as long with
// chunks of 8192 lines, between 0.96 and 1.92.
std::vector<int64_t> line_chunks(const std::vector<BatchReq>& reqs, int slots) {
    const size_t n = reqs.size();
    std::vector<int64_t> best(n, 1), cur(n, 1);
    double best_time = -1.0, longest0 = 0.0;
    for (int step = 0; step < 8; ++step) {
        static const double kBound[8] = {0.0, 0.7, 0.5, 0.35, 0.25, 0.18, 0.12, 0.08};
        const double bound = step == 0 ? 1e300 : kBound[step] * longest0;
        double total = 0.0, longest = 0.0, tiles = 0.0;
        for (size_t i = 0; i < n; ++i) {
            const BatchReq& q = reqs[i];
            cur[i] = 1;
            if (q.bands <= 0 || q.detectors <= 0) continue;
            const int64_t cap = std::max<int64_t>(
                1, std::min<int64_t>(8192, max_chunk_lines(q.detectors, kBatchThreads,
                                                           kBatchUnroll)));
            const int64_t kmin = std::max<int64_t>(1, (q.lines + cap - 1) / cap);
            const double w = (double)std::min<int64_t>(1 << q.log_strip, q.detectors);
            const double row = (double)detector_cost(q, 0);
            // Lines that keep the tile within the bound, but not fewer than
            // cost as much as the LUT strip.
            const double fit = std::max(bound / w - row, row) / 4.0;
            const int64_t k = fit >= (double)q.lines
                                  ? 1
                                  : (int64_t)std::ceil((double)q.lines / std::max(1.0, fit));
            cur[i] = std::max(kmin, std::min<int64_t>(k, std::max<int64_t>(1, q.lines)));
            const double lines = (double)((q.lines + cur[i] - 1) / cur[i]);
            total += (double)q.bands * (double)q.detectors *
                     ((double)q.lines * 4.0 + (double)cur[i] * row);
            longest = std::max(longest, w * (lines * 4.0 + row));
            tiles += (double)q.bands * std::ceil((double)q.detectors / w) * (double)cur[i];
        }
        if (step == 0) longest0 = longest;
        const double t = tiles <= (double)slots ? longest : total / (double)slots + 0.6 * longest;
        if (best_time < 0.0 || t < best_time) {
            best_time = t;
            best = cur;
        }
    }
    return best;
}

// The batch of n requests; every request takes the tile shape *forced when
// it is given (the tuner's candidates), else its batch entry of the plan
// cache, else the plain path's plan fitted to the batch kernel.
rc_status batch_create(const rc_request* reqs, int32_t n, int32_t flags, const rc_plan* forced,
                       rc_batch** out) {
    if (!out || n < 0 || (n > 0 && !reqs)) return RC_EINVAL;
    *out = nullptr;
    // Pass 1, host only: validate every request and the hazards between them.
    const rc_status vs = validate_requests(reqs, n);
    if (vs != RC_OK) return vs;

    // Pass 2: per-request plans and the tile queue.
    const DeviceInfo* di = current_device();
    if (!di) return RC_EHIP;
    const size_t lds_cap = std::min(kBatchLds, di->lds);
    std::vector<BatchReq> hreq;
    std::vector<BatchTile> htile;
    std::vector<int64_t> prefix(1, 0);
    int64_t total_px = 0, total_lut = 0, gather_lut = 0;
    int32_t ntuned = 0, nfused = 0;
    for (int32_t i = 0; i < n; ++i) {
        const rc_request& r = reqs[i];
        const int64_t px = r.lines * r.detectors * (int64_t)r.bands;
        const int64_t rows = (int64_t)r.bands * r.detectors;
        const int64_t lut_n = rows * r.levels;
        BatchReq q;
        std::memset(&q, 0, sizeof q);
        q.coeffs = r.coeffs;
        q.dn = r.dn;
        q.lut = r.lut;
        q.out = r.out;
        q.lines = r.lines;
        q.detectors = r.detectors;
        q.bands = r.bands;
        q.levels = r.levels;
        q.lut_vec = (r.levels % 8 == 0 && ((uintptr_t)r.lut & 15u) == 0) ? 1 : 0;
        if (rows > 0) {
            const int vmax = px > 0 ? max_vec(r.dn, r.out, r.detectors) : 1;
            const int64_t lines_p = std::max<int64_t>(r.lines, 1);
            rc_plan p;
            if (forced) {
                p = *forced;
            } else if (tuned_batch_shape(r.detectors, r.levels, vmax, *di, &p)) {
                ++ntuned;
            } else {
                batch_plan(lines_p, r.detectors, r.bands, r.levels, vmax, *di, &p);
            }
            fit_request_plan(p, r.levels, lds_cap, &q);
            if (q.mode == kGlobal) gather_lut += lut_n;  // read back by the gather
            else ++nfused;                                // never read back
            if (max_chunk_lines(r.detectors, kBatchThreads, kBatchUnroll) < 1)
                return RC_EINVAL;  // lines too wide for 32-bit tile offsets
        }
        hreq.push_back(q);
        const int64_t items =
            (rows > 0 && q.mode == kGlobal) ? rows * (int64_t)((r.levels + 7) / 8) : 0;
        prefix.push_back(prefix.back() + items);
        total_px += px;
        total_lut += lut_n;
    }
    const int slots =
        std::max(1, di->cus) *
        (int)std::max<size_t>(1, std::min<size_t>(kBatchPerCu, di->lds_per_cu / lds_cap));
    // One tile per (band, strip) and line chunk.
    const std::vector<int64_t> chunks = line_chunks(hreq, slots);
    for (int32_t i = 0; i < n; ++i) {
        const BatchReq& q = hreq[i];
        if (q.bands <= 0 || q.detectors <= 0) continue;
        const int64_t ch = std::max<int64_t>(1, (q.lines + chunks[i] - 1) / chunks[i]);
        const int32_t strips = (int32_t)(((int64_t)q.detectors + (1 << q.log_strip) - 1) >>
                                         q.log_strip);
        // A fused request with no lines still gets one tile per strip, which
        // only builds the LUT (the other mode's LUTs come from the build
        // kernel).
        const int64_t nend = (q.lines == 0 && q.fused) ? 1 : q.lines;
        for (int32_t b = 0; b < q.bands; ++b)
            for (int32_t st = 0; st < strips; ++st)
                for (int64_t n0 = 0; n0 < nend; n0 += ch) {
                    BatchTile tl;
                    tl.req = i;
                    tl.band = b;
                    tl.d0 = strip_start(q, st);
                    tl.pad = 0;
                    tl.n0 = n0;
                    tl.n1 = std::min(q.lines, n0 + ch);
                    htile.push_back(tl);
                }
    }
    if (htile.size() > (size_t)INT32_MAX) return RC_EINVAL;
    auto cost = [&](const BatchTile& t) {
        const BatchReq& q = hreq[t.req];
        return std::min<int64_t>(1 << q.log_strip, q.detectors - t.d0) *
               detector_cost(q, t.n1 - t.n0);
    };
    // Tiles of one (request, band, line chunk) are a group: its strips hold
    // neighbouring segments of the same lines, which share cache lines where a
    // line's bytes do not start on a 128-byte boundary. A group goes whole to
    // one XCD's queue, strips in order, so those lines are fetched once into
    // that XCD's L2. Groups are dealt longest first to the least loaded queue
    // and keep that order inside it.
    struct Group {
        int64_t cost = 0;
        size_t first = 0, count = 0;
    };
    std::stable_sort(htile.begin(), htile.end(), [](const BatchTile& a, const BatchTile& b) {
        if (a.req != b.req) return a.req < b.req;
        if (a.band != b.band) return a.band < b.band;
        if (a.n0 != b.n0) return a.n0 < b.n0;
        return a.d0 < b.d0;
    });
    std::vector<Group> groups;
    for (size_t i = 0; i < htile.size(); ++i) {
        const BatchTile& t = htile[i];
        if (i == 0 || t.req != htile[i - 1].req || t.band != htile[i - 1].band ||
            t.n0 != htile[i - 1].n0) {
            Group g;
            g.first = i;
            groups.push_back(g);
        }
        groups.back().count += 1;
        groups.back().cost += cost(t);
    }
    std::stable_sort(groups.begin(), groups.end(),
                     [](const Group& a, const Group& b) { return a.cost > b.cost; });
    std::vector<std::vector<size_t>> qgroups(kBatchQueues);
    int64_t qload[kBatchQueues] = {};
    for (size_t gi = 0; gi < groups.size(); ++gi) {
        int best = 0;
        for (int qi = 1; qi < kBatchQueues; ++qi)
            if (qload[qi] < qload[best]) best = qi;
        qgroups[best].push_back(gi);
        qload[best] += groups[gi].cost;
    }
    std::vector<BatchTile> ordered;
    ordered.reserve(htile.size());
    BatchQueues queues;
    for (int qi = 0; qi < kBatchQueues; ++qi) {
        queues.bound[qi] = (int32_t)ordered.size();
        for (size_t gi : qgroups[qi])
            for (size_t k = 0; k < groups[gi].count; ++k)
                ordered.push_back(htile[groups[gi].first + k]);
    }
    queues.bound[kBatchQueues] = (int32_t)ordered.size();
    htile.swap(ordered);

    rc_batch* bt = new (std::nothrow) rc_batch();
    if (!bt) return RC_ENOMEM;
    const hipError_t dev_err = hipGetDevice(&bt->device);
    if (dev_err != hipSuccess) {
        delete bt;
        return hip_fail(dev_err);
    }
    bt->nreq = n;
    bt->ntiles = (int32_t)htile.size();
    bt->queues = queues;
    bt->build_items = prefix.back();
    bt->cus = di->cus;
    bt->lds = lds_cap;
    bt->use_graph = !(flags & RC_BATCH_NO_GRAPH);
    bt->slots = slots;
    hipError_t e = hipSuccess;
    auto fail = [&](hipError_t err) {
        release(bt);
        return err == hipErrorOutOfMemory ? RC_ENOMEM : hip_fail(err);
    };
    if (n > 0) {
        if ((e = hipMalloc(&bt->d_reqs, sizeof(BatchReq) * n)) != hipSuccess) return fail(e);
        if ((e = hipMalloc(&bt->d_prefix, sizeof(int64_t) * (n + 1))) != hipSuccess) return fail(e);
    }
    if (!htile.empty() &&
        (e = hipMalloc(&bt->d_tiles, sizeof(BatchTile) * htile.size())) != hipSuccess)
        return fail(e);
    if ((e = hipMalloc(&bt->d_counters, kBatchCounters * sizeof(unsigned int))) != hipSuccess)
        return fail(e);
    if ((e = hipStreamCreateWithFlags(&bt->cap, hipStreamNonBlocking)) != hipSuccess)
        return fail(e);
    if (n > 0) {
        if ((e = hipMemcpyAsync(bt->d_reqs, hreq.data(), sizeof(BatchReq) * n,
                                hipMemcpyHostToDevice, bt->cap)) != hipSuccess)
            return fail(e);
        if ((e = hipMemcpyAsync(bt->d_prefix, prefix.data(), sizeof(int64_t) * (n + 1),
                                hipMemcpyHostToDevice, bt->cap)) != hipSuccess)
            return fail(e);
    }
    if (!htile.empty() &&
        (e = hipMemcpyAsync(bt->d_tiles, htile.data(), sizeof(BatchTile) * htile.size(),
                            hipMemcpyHostToDevice, bt->cap)) != hipSuccess)
        return fail(e);
    if ((e = hipMemsetAsync(bt->d_counters, 0, kBatchCounters * sizeof(unsigned int), bt->cap)) !=
        hipSuccess)
        return fail(e);
    if ((e = hipStreamSynchronize(bt->cap)) != hipSuccess) return fail(e);
    if ((e = prepare_batch_kernel(lds_cap)) != hipSuccess) return fail(e);
    if (bt->use_graph) {
        if ((e = hipStreamBeginCapture(bt->cap, hipStreamCaptureModeThreadLocal)) != hipSuccess)
            return fail(e);
        const hipError_t le = enqueue(bt, bt->cap);
        e = hipStreamEndCapture(bt->cap, &bt->graph);
        if (le != hipSuccess) return fail(le);
        if (e != hipSuccess) return fail(e);
        if ((e = hipGraphInstantiate(&bt->exec, bt->graph, nullptr, nullptr, 0)) != hipSuccess)
            return fail(e);
    }
    rc_batch_stats& st = bt->stats;
    st.requests = n;
    st.tiles = bt->ntiles;
    st.slots = bt->slots;
    st.pixels = total_px;
    st.lut_entries = total_lut;
    st.graph = bt->use_graph ? 1 : 0;
    st.tuned = ntuned;
    st.fused = nfused;
    st.lut_gather_entries = gather_lut;
    *out = bt;
    return RC_OK;
}

// Candidate tile shapes of the batch kernel for requests with `levels`
// levels and at most `dmax` detectors: the LDS paths at the widest strip that
// fits the batch's tile budget and narrower ones, the L2 path at two widths
// (pixels per lane follow from the rows, fit_request_plan).
std::vector<rc_plan> batch_candidates(int32_t levels, int32_t dmax, size_t lds_cap, int effort) {
    std::vector<rc_plan> out;
    int wcap = 8;
    while (wcap < dmax && wcap < 1024) wcap <<= 1;
    auto add = [&](int path, int W) {
        if (W < 1 || W > wcap) return;
        rc_plan p;
        std::memset(&p, 0, sizeof p);
        p.path = path;
        p.strip = W;
        p.vec = 1;
        p.threads = kBatchThreads;
        p.unroll = kBatchUnroll;
        p.chunk_lines = 1;
        p.xcd_remap = 1;
        out.push_back(p);
    };
    for (int path : {RC_PATH_DENSE, RC_PATH_PACKED, RC_PATH_LDS}) {
        if (path == RC_PATH_DENSE && levels > kDenseMaxLevels) continue;
        int w0 = 0;
        for (int W = 1024; W >= 8; W >>= 1)
            if (plan_lds_bytes(path, W, levels) <= lds_cap) {
                w0 = std::min(W, wcap);
                break;
            }
        if (!w0) continue;
        for (int k = 0; k < (effort ? 3 : 2); ++k) add(path, w0 >> k);
    }
    for (int W : {64, 128}) add(RC_PATH_L2, W);
    return out;
}

}  // namespace

extern "C" {

rc_status rc_batch_create(const rc_request* reqs, int32_t n, int32_t flags, rc_batch** out) {
    return batch_create(reqs, n, flags, nullptr, out);
}

rc_status rc_batch_tune(const rc_request* reqs, int32_t n, int32_t effort, int32_t* classes,
                        hipStream_t stream) {
    if (classes) *classes = 0;
    if (n < 0 || (n > 0 && !reqs)) return RC_EINVAL;
    const rc_status vs = validate_requests(reqs, n);
    if (vs != RC_OK) return vs;
    const DeviceInfo* di = current_device();
    if (!di) return RC_EHIP;
    const size_t lds_cap = std::min(kBatchLds, di->lds);
    // Shape classes: (levels, ceil(log2 detectors), vector width), over the
    // requests that have pixels.
    struct Cls {
        int32_t levels;
        int dclass;
        int vmax;
        int32_t dmax;
        std::vector<rc_request> reqs;
    };
    std::vector<Cls> cls;
    for (int32_t i = 0; i < n; ++i) {
        const rc_request& r = reqs[i];
        if (r.lines <= 0 || r.detectors <= 0 || r.bands <= 0) continue;
        const int vmax = max_vec(r.dn, r.out, r.detectors);
        int dc = 0;
        while (((int64_t)1 << dc) < r.detectors) ++dc;
        auto it = std::find_if(cls.begin(), cls.end(), [&](const Cls& c) {
            return c.levels == r.levels && c.dclass == dc && c.vmax == vmax;
        });
        if (it == cls.end()) {
            cls.push_back(Cls{r.levels, dc, vmax, 0, {}});
            it = cls.end() - 1;
        }
        it->dmax = std::max(it->dmax, r.detectors);
        it->reqs.push_back(r);
    }
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    rc_status st = e == hipSuccess ? RC_OK : hip_fail(e);
    const int reps = 3;
    int32_t done = 0;
    for (const Cls& c : cls) {
        if (st != RC_OK) break;
        float best = 1e30f;
        rc_plan best_p{};
        // The shape rc_batch_create would take without a batch entry comes
        // first; another candidate replaces the best so far only if it is at
        // least 2 % faster (timings of one class's requests vary by about
        // that much, and a narrower strip chosen on noise makes neighbouring
        // strips fetch more shared lines).
        std::vector<rc_plan> cands;
        {
            const rc_request& r0 = c.reqs.front();
            rc_plan h;
            const int64_t lines_p = std::max<int64_t>(r0.lines, 1);
            batch_plan(lines_p, r0.detectors, r0.bands, r0.levels, c.vmax, *di, &h);
            cands.push_back(h);
            for (const rc_plan& x : batch_candidates(c.levels, c.dmax, lds_cap, effort))
                cands.push_back(x);
        }
        for (const rc_plan& cand : cands) {
            rc_batch* b = nullptr;
            const rc_status cs = batch_create(c.reqs.data(), (int32_t)c.reqs.size(),
                                              RC_BATCH_NO_GRAPH, &cand, &b);
            if (cs == RC_EINVAL) continue;  // not runnable for this class
            if (cs != RC_OK) {
                st = cs;
                break;
            }
            float ms = 0.f;
            if ((e = enqueue(b, stream)) == hipSuccess &&  // warm-up run
                (e = hipEventRecord(e0, stream)) == hipSuccess) {
                for (int r = 0; r < reps && e == hipSuccess; ++r) e = enqueue(b, stream);
                if (e == hipSuccess) e = hipEventRecord(e1, stream);
                if (e == hipSuccess) e = hipEventSynchronize(e1);
                if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
            }
            // The runs must be over before the batch's tables are freed.
            const hipError_t se = hipStreamSynchronize(stream);
            if (e == hipSuccess) e = se;
            release(b);
            if (e != hipSuccess) {
                st = hip_fail(e);
                break;
            }
            ms /= reps;
            if (ms < (best < 1e30f ? best * 0.98f : best)) {
                best = ms;
                best_p = cand;
            }
        }
        if (st == RC_OK && best < 1e30f) {
            store_batch_shape(c.dmax, c.levels, c.vmax, *di, best_p, best * 1000.0);
            ++done;
        }
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (classes) *classes = done;
    return st;
}

rc_status rc_batch_run(rc_batch* b, hipStream_t stream) {
    if (!b) return RC_EINVAL;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e);
    if (dev != b->device) return RC_EINVAL;
    e = b->use_graph ? hipGraphLaunch(b->exec, stream) : enqueue(b, stream);
    return e == hipSuccess ? RC_OK : hip_fail(e);
}

rc_status rc_batch_info(const rc_batch* b, rc_batch_stats* st) {
    if (!b || !st) return RC_EINVAL;
    *st = b->stats;
    return RC_OK;
}

void rc_batch_destroy(rc_batch* b) { release(b); }

}  // extern "C"
