// The library's host side (hough_host.hip) with launches that are written down
// instead of made: one JSON object per launch or limit that it sets.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <string>

#include "hough_internal.h"
#include "hough_tw.h"

namespace {
std::string log_text;
void note(const char *fmt, ...) {
    char line[512];
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(line, sizeof line, fmt, ap);
    va_end(ap);
    log_text += line;
    log_text += "\n";
}
}  // namespace

extern "C" const char *launches() {   // since the last call
    static std::string out;
    out.swap(log_text);
    log_text.clear();
    return out.c_str();
}
extern "C" void set_memory(size_t bytes) { memory_left = bytes; }

namespace hough {

// as in hough_kernels.hip and hough_cf.hip
int find_lds_extra(int threads, int hcap, int pkeep) { return 4 * hcap + 8 * (pkeep + hcap) + 4 * threads; }
int sweep_lds_bytes(int threads, int pitch) { return (threads / 64) * pitch * 4 + 4 * threads; }
int band_lds_bytes(int pitch, int hits) {
    return ((hits * 8 + 15) & ~15) + 4 * (4 * 3 * (pitch / 2)) + 4 * (4 * 3 * 128) + 8 * (4 * 512) + 4 * kBandThreads;
}
int cf_lds_bytes(int c, int f, int) { return ((4 * c + 15) & ~15) + ((4 * f + 15) & ~15) + 8 * kCfStage + 16 * 16 + 16; }

hipError_t set_find_lds_limit(int threads, int bytes) {
    note("{\"limit\": \"find\", \"threads\": %d, \"bytes\": %d}", threads, bytes);
    return hipSuccess;
}
hipError_t set_tw_lds_limit(int threads, int bytes) {
    note("{\"limit\": \"tw\", \"threads\": %d, \"bytes\": %d}", threads, bytes);
    return hipSuccess;
}
hipError_t set_cf_lds_limit(int threads, int bytes) {
    note("{\"limit\": \"cf\", \"threads\": %d, \"bytes\": %d}", threads, bytes);
    return hipSuccess;
}
hipError_t set_tw_cf_lds_limit(int threads, int bytes) {
    note("{\"limit\": \"tw_cf\", \"threads\": %d, \"bytes\": %d}", threads, bytes);
    return hipSuccess;
}
hipError_t set_sweep_lds_limit(int threads, int bytes) {
    note("{\"limit\": \"sweep\", \"threads\": %d, \"bytes\": %d}", threads, bytes);
    return hipSuccess;
}
hipError_t set_band_lds_limit(int bytes) {
    note("{\"limit\": \"band\", \"threads\": %d, \"bytes\": %d}", kBandThreads, bytes);
    return hipSuccess;
}
hipError_t set_dump_lds_limit(int bytes) {
    note("{\"limit\": \"dump\", \"threads\": 0, \"bytes\": %d}", bytes);
    return hipSuccess;
}
hipError_t cf_blocks_per_cu(int threads, int lds, int *blocks) {   // four waves per SIMD, 160 KB
    *blocks = std::min(1024 / threads, (160 << 10) / (lds + kStaticLds));
    return hipSuccess;
}
hipError_t find_blocks_per_cu(int threads, bool argmax, int lds, int *blocks, int *most) {
    cf_blocks_per_cu(threads, lds, blocks);
    *most = threads == 256 && argmax ? *blocks + 1 : *blocks;   // some kernel with fewer registers
    return hipSuccess;
}

hipError_t launch_find(const FindArgs &a, int threads, int lds, hipStream_t) {
    note("{\"launch\": \"find\", \"threads\": %d, \"lds\": %d, \"rows\": %d, \"stream_ok\": %d, \"hs_cap\": %d, \"events\": %d, "
         "\"ordered\": %d, \"slots\": %d, \"split\": %d}",
         threads, lds, a.tile_rows, a.stream_ok, a.hs_cap, a.n_events, a.order != nullptr, a.pool_slots, a.g_hs != nullptr);
    return hipSuccess;
}
hipError_t launch_find_cf(const FindArgs &, int threads, int lds, hipStream_t) {
    note("{\"launch\": \"find_cf\", \"threads\": %d, \"lds\": %d}", threads, lds);
    return hipSuccess;
}
hipError_t launch_sweep(const FindArgs &a, int threads, int groups, hipStream_t) {
    note("{\"launch\": \"sweep\", \"threads\": %d, \"groups\": %d, \"hs_cap\": %d}", threads, groups, a.hs_cap);
    return hipSuccess;
}
hipError_t launch_band(const FindArgs &, int nwf, int lds, hipStream_t) {
    note("{\"launch\": \"band\", \"waves\": %d, \"lds\": %d}", nwf, lds);
    return hipSuccess;
}
hipError_t launch_order(const int64_t *, int32_t n, int32_t *, hipStream_t) {
    note("{\"launch\": \"order\", \"events\": %d}", n);
    return hipSuccess;
}
hipError_t launch_order_pick(const FindArgs &a, int32_t *, Pick *, int64_t hits, hipStream_t) {
    note("{\"launch\": \"order_pick\", \"events\": %d, \"hits\": %lld}", a.n_events, (long long)hits);
    return hipSuccess;
}
hipError_t launch_picked(const FindArgs &a, int threads, int lds, bool defer, hipStream_t) {
    note("{\"launch\": \"picked\", \"threads\": %d, \"lds\": %d, \"rows\": %d, \"hs_cap\": %d, \"events\": %d, \"slots\": %d, \"defer\": %d}",
         threads, lds, a.tile_rows, a.hs_cap, a.n_events, a.pool_slots, defer);
    return threads == 512 || (threads == 256 && defer) ? hipSuccess : 1;
}
hipError_t launch_list(const FindArgs &a, Pick *, int groups, int threads, int lds, hipStream_t) {
    note("{\"launch\": \"list\", \"threads\": %d, \"lds\": %d, \"rows\": %d, \"groups\": %d, \"stream_ok\": %d, \"split\": %d}", threads, lds,
         a.tile_rows, groups, a.stream_ok, a.g_hs != nullptr);
    return threads == 1024 ? hipSuccess : 1;   // the kernels there are
}
hipError_t launch_compact(const CompactArgs &a, hipStream_t) {
    note("{\"launch\": \"compact\", \"ordered\": %d}", a.ordered);
    return hipSuccess;
}
hipError_t launch_clear_workspace(long long *, int32_t *, int32_t *, int64_t, int32_t *, int32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_dump(const DumpArgs &, int, hipStream_t) { return hipSuccess; }
hipError_t launch_set_offsets(int64_t *, int64_t, hipStream_t) { return hipSuccess; }
hipError_t lds_atomic_rate(int, hipStream_t, int, double *) { return hipSuccess; }

}  // namespace hough
