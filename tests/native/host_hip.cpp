// The HIP runtime and the kernel launchers over host memory, so that the host
// side of libmvf runs in a process without a GPU: kernels do nothing, copies
// are made at once, and every call that allocates, records or launches is
// noted with the device that was current in the calling thread.  Work on a
// stream that nothing orders after all the earlier work on the others is noted
// too: streams, events and the host carry vector clocks; no stream waits for the
// null stream (a caller's are non-blocking), and hipMemset does not wait for
// its clear.  The launchers keep the kernels' books: the counts that a kernel
// appends to must be zero when it starts, and a raycast must find an order that
// no other raycast has used.  A launch can be made to fail.
#include <hip/hip_runtime.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <string>

#include "mvf.h"
#include "mvf_internal.h"

namespace {
thread_local int g_device = 0;
int g_expect = -1;          // device that all device work belongs on (-1: not checked)
std::string g_elsewhere;    // names of calls made while another device was current
int g_allocs = 0;           // device allocations and frees

typedef std::map<void*, long> Clock;   // stream -> work on it that is known to be done
void join(Clock& a, const Clock& b)
{
    for (auto& kv : b) a[kv.first] = std::max(a[kv.first], kv.second);
}
Clock g_host, g_issued;
std::map<void*, Clock> g_stream, g_event;
std::string g_unordered;

int work(const char* name)
{
    if (g_expect >= 0 && g_device != g_expect) g_elsewhere += std::string(name) + " ";
    return 0;
}

std::string g_fail;         // the launch of that name fails, once
std::string g_stale;        // counts that were not zero, orders that were not made
std::map<const void*, bool> g_ordered;

int work(const char* name, void* stream)
{
    if (g_fail == name) {
        g_fail.clear();
        return (int)hipErrorLaunchFailure;
    }
    Clock& seen = g_stream[stream];
    join(seen, g_host);
    bool after_all = true;
    for (auto& kv : g_issued) after_all = after_all && (kv.first == stream || seen[kv.first] >= kv.second);
    if (!after_all) g_unordered += std::string(name) + " ";
    seen[stream] = ++g_issued[stream];
    return work(name);
}
}  // namespace

extern "C" {
void t_expect(int device) { g_expect = device; g_elsewhere.clear(); }
const char* t_elsewhere() { return g_elsewhere.c_str(); }
int t_allocs() { return g_allocs; }
void t_set_device(int device) { g_device = device; }
void* t_stream()
{
    hipStream_t s;
    hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
    return s;
}
void t_watch() { g_unordered.clear(); g_stale.clear(); }
const char* t_stale() { return g_stale.c_str(); }
void t_fail(const char* name) { g_fail = name; }
int t_failed() { return g_fail.empty(); }
const char* t_unordered() { return g_unordered.c_str(); }

hipError_t hipGetDeviceCount(int* n) { *n = 2; return hipSuccess; }
hipError_t hipSetDevice(int d) { g_device = d; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { join(g_host, g_issued); return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipMalloc(void** p, size_t n) { ++g_allocs; *p = calloc(1, n ? n : 1); return (hipError_t)work("hipMalloc"); }
hipError_t hipFree(void* p) { ++g_allocs; free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n ? n : 1); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { join(g_host, g_stream[s]); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t stream)
{
    memcpy(d, s, n);
    return (hipError_t)work("hipMemcpyAsync", stream);
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k)
{
    hipMemcpyAsync(d, s, n, k, nullptr);
    return hipStreamSynchronize(nullptr);
}
hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return (hipError_t)work("hipMemset", nullptr); }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)malloc(1); return (hipError_t)work("hipEventCreate"); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { g_event.erase(e); free((void*)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    g_event[e] = g_host;
    join(g_event[e], g_stream[s]);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { join(g_host, g_event[e]); return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)malloc(1); return (hipError_t)work("hipStreamCreate"); }
hipError_t hipStreamDestroy(hipStream_t s)
{
    g_stream.erase(s);
    g_issued.erase(s);
    free((void*)s);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { join(g_stream[s], g_event[e]); return hipSuccess; }
}

namespace mvf {
int launch_frame_prep(const PrepItem*, int, int, int, void* s, const void* tsrc, void* tdst, size_t tbytes)
{
    const int e = work("frame_prep", s);
    if (!e && tsrc) memcpy(tdst, tsrc, tbytes);
    return e;
}
int launch_volume_init(DevVolume, void* s) { return work("volume_init", s); }
int launch_ztable(const IntegrateLaunch& L, int, void* s)
{
    const int e = work("ztable", s);
    if (e || !L.list_count) return e;
    const int par = L.hdr->list_parity;
    if (L.list_count[par]) g_stale += "list ";
    L.list_count[par] = 1;
    L.list_count[par ^ 1] = 0;
    return 0;
}
void ordered(const TileOrder& o)
{
    if (o.tiles > 0) g_ordered[o.order] = true;
}
void collect(const LaunchHeader* hdr, const RayBounds& rb)
{
    for (int v = 0; v < hdr->nvol; ++v) {
        uint32_t& n = rb.counts[(size_t)hdr->rb_parity * rb.cap + v];
        if (n) g_stale += "footprints ";
        n = 1;
    }
}
int launch_integrate(const IntegrateLaunch& L, int, void* s, void*, void*)
{
    const int e = work("integrate", s);
    if (!e) ordered(L.order);
    return e;
}
int launch_raycast(const RaycastLaunch& L, int, void* s, void*, void*)
{
    const int e = work("raycast", s);
    if (!e && !g_ordered[L.tile_order]) g_stale += "order ";
    g_ordered[L.tile_order] = false;
    return e;
}
int launch_column_flags(DevVolume, void* s) { return work("column_flags", s); }
int launch_brick_distance(const LaunchHeader* hdr, const DevVolume*, const int32_t*, int, int bricks, void* s,
                          const DevFrame* frames, RayBounds rb)
{
    if (bricks <= 0) return 0;
    const int e = work("brick_distance", s);
    if (!e && frames && rb.entries) collect(hdr, rb);
    return e;
}
int launch_ray_bounds_collect(const LaunchHeader* hdr, const DevVolume*, const int32_t*, const DevFrame*, RayBounds rb, int,
                              void* s)
{
    const int e = work("ray_bounds_collect", s);
    if (!e) collect(hdr, rb);
    return e;
}
int launch_ray_bounds_merge(const LaunchHeader* hdr, const DevFrame*, const int32_t*, const int32_t*, const int32_t*,
                            RayBounds rb, int, int, int, void* s, TileOrder order)
{
    const int e = work("ray_bounds_merge", s);
    if (e) return e;
    std::fill_n(rb.counts + (size_t)(1 - hdr->rb_parity) * rb.cap, rb.cap, 0u);
    ordered(order);
    return 0;
}
int launch_swap_copy(const void* src, void* dst, size_t bytes, void* s)
{
    memcpy(dst, src, bytes);
    return work("swap_copy", s);
}
int launch_read_plane(DevVolume, int plane, uint32_t, uint32_t n, void* out, void* s)
{
    memset(out, 0, (size_t)n * (plane == 1 ? 2 : 4));
    return work("read_plane", s);
}
int launch_import(DevVolume, const float*, const uint16_t*, const uint32_t*, bool, void* s) { return work("import", s); }
size_t extract_buffer_bytes(size_t nbricks) { return 64 * nbricks; }
ExtractBuffers extract_buffers(void*, size_t, long long* total)
{
    ExtractBuffers B{};
    B.total = total;
    return B;
}
int launch_extract(DevVolume, const ExtractBuffers&, float*, float*, int32_t*, long long, void* s) { return work("extract", s); }
int launch_fill_u64(unsigned long long* p, int n, unsigned long long value, void* s)
{
    const int e = work("fill", s);
    if (!e) std::fill(p, p + n, value);
    return e;
}
int launch_placement_clear(unsigned long long*, int, int*, void* s) { return work("placement_clear", s); }
int launch_placement_count(const PlacementCount&, PlacementCells* out, void* s)
{
    out->n = out->overflow = 0;
    return work("placement_count", s);
}
int launch_track_smooth(const float*, int, int, int, float, float*, void* s) { return work("track_smooth", s); }
int launch_track_down(const float*, int, int, int, float, float*, void* s) { return work("track_down", s); }
int launch_track_maps(TrackMaps, void* s) { return work("track_maps", s); }
int track_blocks(int, int) { return 1; }
int launch_icp_step(const TrackLaunch&, int, TrackState*, void* s) { return work("icp_step", s); }
int diffray_scratch_init(int) { return 0; }
double* diffray_scratch(int) { return nullptr; }
int diffray_partials_needed(int, int) { return 1; }
int launch_diffray_backward(DiffVolume, const float*, float, float, float, float, int, int, RayParams, const float*,
                            const int32_t*, float*, double*, int, double*, void* s) { return work("diffray_backward", s); }
}  // namespace mvf
