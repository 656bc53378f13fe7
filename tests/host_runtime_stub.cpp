// A stand-in for the HIP runtime and the kernel launches, so the host side of
// the library (arena_host.cpp) runs on a machine without a GPU.  "Device"
// memory is host memory from malloc; copies happen at once, except while the
// stream is captured, when they are only counted (a graph would run them at a
// replay).  Freed blocks are remembered: a launch whose arguments point into
// one, or whose split caches are smaller than its blocks need, is counted as a
// fault.  The estimate's launch copies pending contention factors as its
// prologue kernel does.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <vector>

#include "arena_internal.h"

namespace {

std::map<char*, size_t> live;
bool capturing = false;
int n_allocs = 0, n_frees = 0, n_faults = 0, n_launches = 0, n_recorded_copies = 0;
arena::EstimateArgs last{};
std::vector<float> seen_kappa;       // contention factors the last launch outside a capture read

bool in_live(const void* p, size_t bytes)
{
    auto it = live.upper_bound((char*)p);
    if (it == live.begin()) return false;
    --it;
    return (char*)p >= it->first && (char*)p + bytes <= it->first + it->second;
}

}  // namespace

extern "C" {

hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
const char* hipGetErrorString(hipError_t e)
{
    return e == hipErrorStreamCaptureUnsupported ? "operation not permitted when stream is capturing" : "error";
}
hipError_t hipMalloc(void** p, size_t n)
{
    *p = std::malloc(n);
    live[(char*)*p] = n;
    ++n_allocs;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    // the address stays taken, so that no later block gets it
    if (p) n_frees += (int)live.erase((char*)p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    if (capturing) ++n_recorded_copies;
    else std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return capturing ? hipErrorStreamCaptureUnsupported : hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)std::malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { std::free((void*)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s)
{
    *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}

void stub_capture(int on) { capturing = on != 0; }
int stub_allocs() { return n_allocs; }
int stub_frees() { return n_frees; }
int stub_faults() { return n_faults; }
int stub_launches() { return n_launches; }
int stub_recorded_copies() { return n_recorded_copies; }
int stub_blocks() { return last.n_blocks; }
int stub_parts() { return last.n_parts; }
float stub_kappa(int i) { return seen_kappa[(size_t)i]; }
long long stub_live_bytes()
{
    long long n = 0;
    for (const auto& b : live) n += (long long)b.second;
    return n;
}
// Would a replay of the launch recorded last touch freed memory?
int stub_last_dangles()
{
    const size_t items = (size_t)last.n_items, nc = (size_t)last.n_counts;
    return !(in_live(last.pure_cuts, (size_t)last.n_blocks * arena::kPureCutBytes) &&
             in_live(last.layer_offset, 4 * ((size_t)last.n_jobs + 1)) && in_live(last.batch, 4 * (size_t)last.n_jobs) &&
             in_live(last.item_order, 4 * items) && in_live(last.count_order, 4 * nc) &&
             in_live(last.counts, 4 * nc) && in_live(last.kappa, 4 * nc * (size_t)last.n_types) &&
             in_live(last.types, sizeof(arena::TypeDev) * (size_t)last.n_types) &&
             in_live(last.queue, 8 * arena::kQueues) && in_live(last.counters, 8 * arena::kNumCounters));
}

}  // extern "C"

namespace arena {

hipError_t launch_estimate(const EstimateArgs& args, hipStream_t)
{
    last = args;
    ++n_launches;
    n_faults += stub_last_dangles();
    const int nk = args.n_types * args.n_counts;
    if (!capturing) {
        if (args.kappa_src) std::memcpy(args.kappa, args.kappa_src, sizeof(float) * (size_t)nk);
        seen_kappa.assign(args.kappa, args.kappa + nk);
    }
    return hipSuccess;
}

hipError_t launch_proxy(const ProxyArgs& args, hipStream_t)
{
    ++n_launches;
    if (!capturing) seen_kappa.assign(args.kappa, args.kappa + args.n_types * args.n_counts);
    return hipSuccess;
}

hipError_t scratch_address(int, void** out)
{
    static std::vector<char> scratch(kNoallocScratchBytes);
    *out = scratch.data();
    return hipSuccess;
}

hipError_t launch_schedule(const SchedArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_zero_counters(unsigned long long* p, int n, hipStream_t)
{
    if (!capturing) std::memset(p, 0, sizeof(*p) * (size_t)n);
    return hipSuccess;
}
hipError_t launch_validate(const ValidateArgs&, hipStream_t) { return hipSuccess; }

}  // namespace arena
