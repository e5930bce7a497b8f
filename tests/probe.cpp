// Host-side choices of librc (launch shapes, plans, strips) by their internal names, for tests
// that need no GPU. Each line of standard input is a command; each gives one line of output.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <iostream>
#include <sstream>
#include <string>

#include "batch.h"
#include "kernels.h"
#include "runtime.h"

using namespace rc;

// demosaic <bilinear|gradient> images H W sectors: rows per band.
static void demosaic(std::istringstream& in) {
    std::string method;
    int images, H, W, sectors;
    in >> method >> images >> H >> W >> sectors;
    const int64_t band = method == "bilinear"
                             ? demosaic_band(images, H, W, sectors != 0, 256)
                             : demosaic_gradient_band(images, H, W, sectors != 0, 256);
    std::printf("%lld\n", (long long)band);
}

static DeviceInfo mi355x() {
    DeviceInfo di;
    di.cus = 256;
    di.xcds = 8;
    di.lds = di.lds_per_cu = 160 * 1024;
    di.arch = "probe";
    return di;
}

static bool runs(const rc_plan& p, int64_t N, int D, int B, int L, int vmax, const DeviceInfo& di,
                 bool wide = false) {
    ApplyParams a{};
    size_t lds = 0;
    return check_plan(p, N, D, B, L, vmax, di, &a, &lds, wide) == RC_OK;
}

// plan B N D L dn_offset out_offset (bytes; -1: in place): whether the plan rc_correct takes for
// the shape can run; whether power-of-two strips (pow2_plan) or, where those are LDS strips, one
// equal tile per CU (balanced_tiling) can; whether the plan can run as it is.
static void plan(std::istringstream& in) {
    int64_t N;
    int B, D, L, dn_off, out_off;
    in >> B >> N >> D >> L >> dn_off >> out_off;
    const DeviceInfo di = mi355x();
    const uint16_t* dn = (const uint16_t*)(uintptr_t)((1ull << 40) + dn_off);
    const uint16_t* out =
        out_off < 0 ? dn : (const uint16_t*)(uintptr_t)((1ull << 45) + out_off);
    const int vmax = max_vec(dn, out, D, 8);
    rc_plan p, w;
    default_plan(N, D, B, L, vmax, di, &p, dn == out, on_sectors(dn, out));
    w = p;
    const bool ok = (vmax < 8 && widen_plan(dn, out, D, &w) && runs(w, N, D, B, L, vmax, di, true)) ||
                    runs(p, N, D, B, L, vmax, di);
    rc_plan q;
    pow2_plan(N, D, B, L, vmax, di, &q);
    const bool pow2 = runs(q, N, D, B, L, vmax, di);
    const bool lds = q.path != RC_PATH_L2;
    std::memset(&q, 0, sizeof q);
    q.path = L >= 512 ? RC_PATH_PACKED : RC_PATH_LDS;
    q.vec = std::min(vmax, 2);
    q.threads = 256;
    q.unroll = 8;
    q.xcd_remap = q.lane_map = 1;
    const int wmax = widest_strip(q.path, L, di.lds);
    const bool even = lds && wmax >= 16 &&
                      balanced_tiling(N, D, B, q.vec, wmax, di.cus, q.threads, q.unroll, &q.strips,
                                      &q.strip, &q.chunk_lines) &&
                      runs(q, N, D, B, L, vmax, di);
    std::printf("%d %d %d %d\n", ok, pow2, even, runs(p, N, D, B, L, vmax, di));
}

// choice B N D L dn_offset out_offset: rc_correct's plan: path strip strips vec threads chunk_lines
// nontemporal.
static void choice(std::istringstream& in) {
    int64_t N;
    int B, D, L, dn_off, out_off;
    in >> B >> N >> D >> L >> dn_off >> out_off;
    const uint16_t* dn = (const uint16_t*)(uintptr_t)((1ull << 40) + dn_off);
    const uint16_t* out =
        out_off < 0 ? dn : (const uint16_t*)(uintptr_t)((1ull << 45) + out_off);
    rc_plan p;
    default_plan(N, D, B, L, max_vec(dn, out, D, 8), mi355x(), &p, dn == out, on_sectors(dn, out));
    std::printf("%d %d %d %d %d %d %d\n", p.path, p.strip, p.strips, p.vec, p.threads,
                p.chunk_lines, p.nontemporal);
}

// launch B N D L dn_offset out_offset: pixels per lane that rc_correct launches with.
static void launch(std::istringstream& in) {
    int64_t N;
    int B, D, L, dn_off, out_off;
    in >> B >> N >> D >> L >> dn_off >> out_off;
    const DeviceInfo di = mi355x();
    const uint16_t* dn = (const uint16_t*)(uintptr_t)((1ull << 40) + dn_off);
    const uint16_t* out =
        out_off < 0 ? dn : (const uint16_t*)(uintptr_t)((1ull << 45) + out_off);
    rc_plan p;
    ApplyParams a{};
    size_t lds = 0;
    default_plan(N, D, B, L, max_vec(dn, out, D, 8), di, &p, dn == out, on_sectors(dn, out));
    const bool ok = launched_plan(dn, out, N, D, B, L, di, &p, &a, &lds) == RC_OK;
    std::printf("%d\n", ok ? p.vec : 0);
}

// strips D L path W in_place: pixels per lane of a batch request with strips planned W wide, then
// first detector and width of each strip.
static void strips(std::istringstream& in) {
    rc_plan p;
    std::memset(&p, 0, sizeof p);
    BatchReq q;
    std::memset(&q, 0, sizeof q);
    int in_place;
    in >> q.detectors >> q.levels >> p.path >> p.strip >> in_place;
    p.vec = 1;
    q.dn = (const uint16_t*)(uintptr_t)(1ull << 40);
    q.out = in_place ? (uint16_t*)q.dn : (uint16_t*)(uintptr_t)(1ull << 45);
    fit_request_plan(p, q.levels, kBatchLds, &q);
    std::printf("%d", q.vec);
    const int W = 1 << q.log_strip;
    for (int s = 0; s * W < q.detectors; ++s) {
        const int d0 = strip_start(q, s);
        std::printf(" %d %d", d0, strip_width(q, d0));
    }
    std::printf("\n");
}

// tune B N D L dn_offset: number of rc_tune's candidates, and of different plans they run.
static void tune(std::istringstream& in) {
    int64_t N;
    int B, D, L, dn_off;
    in >> B >> N >> D >> L >> dn_off;
    const DeviceInfo di = mi355x();
    const uint16_t* dn = (const uint16_t*)(uintptr_t)((1ull << 40) + dn_off);
    const uint16_t* out = (const uint16_t*)(uintptr_t)(1ull << 45);
    std::vector<std::string> runs;
    const std::vector<rc_plan> cands = tune_candidates(dn, out, N, D, B, L, di, 1);
    for (rc_plan p : cands) {
        ApplyParams a{};
        size_t lds = 0;
        if (launched_plan(dn, out, N, D, B, L, di, &p, &a, &lds) == RC_OK)
            runs.push_back(std::string((const char*)&p, sizeof p));
    }
    std::sort(runs.begin(), runs.end());
    const size_t distinct = std::unique(runs.begin(), runs.end()) - runs.begin();
    std::printf("%zu %zu\n", cands.size(), distinct);
}

// tuned B N D L dn_offset in_place: whether an entry of the plan cache serves the images.
static void tuned(std::istringstream& in) {
    int64_t N;
    int B, D, L, dn_off, in_place;
    in >> B >> N >> D >> L >> dn_off >> in_place;
    const uint16_t* dn = (const uint16_t*)(uintptr_t)((1ull << 40) + dn_off);
    const uint16_t* out = in_place ? dn : (const uint16_t*)(uintptr_t)((1ull << 45) + dn_off);
    rc_plan p;
    std::printf("%d\n", tuned_plan_for(dn, out, N, D, B, L, mi355x(), &p));
}

int main() {
    std::string line, cmd;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        in >> cmd;
        if (cmd == "demosaic") demosaic(in);
        else if (cmd == "plan") plan(in);
        else if (cmd == "strips") strips(in);
        else if (cmd == "choice") choice(in);
        else if (cmd == "launch") launch(in);
        else if (cmd == "tune") tune(in);
        else if (cmd == "tuned") tuned(in);
        else return 1;
        std::fflush(stdout);
    }
    return 0;
}
