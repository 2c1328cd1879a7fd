// llp_host.h - host-side plumbing shared by the C ABI entry points: error
// reporting, option defaults, per-device properties, workspace carving and
// the pinned readback buffer.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <string>

#include "../../include/llp.h"

namespace llp {

// thread-local message for llp_last_error()
void set_error(const char* fmt, ...);
int fail(int status, const char* fmt, ...);

// returns LLP_E_HIP with a message if e != hipSuccess
int hip_check(hipError_t e, const char* what);
#define LLP_HIP(call)                                          \
    do {                                                       \
        int _s = ::llp::hip_check((call), #call);              \
        if (_s) return _s;                                     \
    } while (0)

struct DeviceInfo {
    int device;
    int cus;
    int max_threads;
    size_t lds_per_block;
    std::string arch;
};
const DeviceInfo& device_info();

// Autotuner records (tune.cpp), per (architecture, CU count, kind, size
// class = floor(log2(size))) of the current device.
int size_class(long long size);
void tune_record(int kind, long long size, int block, int chunk);
bool tune_lookup(int kind, long long size, int* block, int* chunk);   // own class, else the nearest
bool tune_last(int kind, int* block, int* chunk);                      // the most recent record
void tune_clear();

// copy of opts with defaults filled in
llp_opts opts_or_default(const llp_opts* o);

// Workspace carving: a bump allocator over a caller-provided or
// library-owned device buffer (256-byte aligned pieces).
struct Carver {
    char* base;
    size_t cap;
    size_t used = 0;
    bool measure_only;
    template <class T>
    T* take(size_t count) {
        size_t bytes = (count * sizeof(T) + 255) & ~(size_t)255;
        size_t at = used;
        used += bytes;
        if (measure_only || used > cap) return nullptr;
        return reinterpret_cast<T*>(base + at);
    }
};

// Resolve the workspace for a solve needing `bytes`: the caller's buffer
// (LLP_E_WORKSPACE if too small) or a library-owned one (grown on demand,
// per device).  *out receives the device pointer.
int get_workspace(const llp_opts& o, size_t bytes, void** out);

// Small pinned host buffer per thread and device, for status readback.
void* pinned_scratch(size_t bytes);

// Workspace of a knapsack (knapsack.hip): a header, then the rows of the groups
// the items are split into and of their merges (2 KN_GROUPS rows at most).
// A workspace of the header alone is enough for a solve that is not split.
constexpr int KN_MAX_W = 16383;
constexpr size_t KN_HEADER_BYTES = 256;
constexpr int KN_GROUPS = 32;
inline size_t knap_stride(int64_t W) { return ((size_t)W + 4) & ~(size_t)3; }   // words per row

// Groups (a power of two) the items of one knapsack are split into: the count
// whose estimated time is least.  Measured on an MI355X, in ns: 290 +
// 0.026 W per item of a group's row sweep, 9000 per level of merges (launch
// and latency) and 4000 for the finishing launch, 5.6e-5 W^2 per merge.  So 64
// items at W = 256 stay whole (33 us, 36 as two groups), 256 at W = 4000 take
// 8 groups (65 us, 115 whole), 4000 at W = 6400 take 32 (195 us, 2049 whole)
// and 4000 at W = 16383 take 16 (455 us, 2736 whole, 599 as 32).
inline int knap_groups(int64_t items, int64_t W) {
    int best = 1;
    int64_t best_ns = INT64_MAX;
    for (int k = 0; (1 << k) <= KN_GROUPS; ++k) {
        const int64_t ns = (items >> k) * (290 + W * 26 / 1000) + (k ? 4000 + 9000 * k : 0) +
                           ((1 << k) - 1) * (W * W / 17857);
        if (ns < best_ns) {
            best_ns = ns;
            best = 1 << k;
        }
    }
    return best;
}
inline size_t knap_bytes(int groups, int64_t W) {
    return KN_HEADER_BYTES + (groups > 1 ? (size_t)2 * groups * knap_stride(W) * 4 : 0);
}
// What a solve of these sizes can use; the header for sizes that it refuses.
inline size_t knap_workspace_bytes(int64_t items, int64_t W) {
    if (items < 0 || items > INT32_MAX || W < 0 || W > KN_MAX_W) return KN_HEADER_BYTES;
    return knap_bytes(knap_groups(items, W), W);
}

// Wait for the stream and read `bytes` from device pointer src into dst via the
// pinned scratch buffer.
int readback(hipStream_t s, const void* src, void* dst, size_t bytes);

}  // namespace llp
