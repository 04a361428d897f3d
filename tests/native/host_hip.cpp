// The HIP runtime and the kernel launchers over host memory, so that the host
// side of libmvf runs in a process without a GPU: kernels do nothing, copies
// are made at once, and every call that allocates, records or launches is
// noted with the device that was current in the calling thread.
#include <hip/hip_runtime.h>
#include <stdlib.h>
#include <string.h>

#include <string>

#include "mvf.h"
#include "mvf_internal.h"

namespace {
thread_local int g_device = 0;
int g_expect = -1;          // device that all device work belongs on (-1: not checked)
std::string g_elsewhere;    // names of calls made while another device was current
int g_allocs = 0;           // device allocations and frees

int work(const char* name)
{
    if (g_expect >= 0 && g_device != g_expect) g_elsewhere += std::string(name) + " ";
    return 0;
}
}  // namespace

extern "C" {
void t_expect(int device) { g_expect = device; g_elsewhere.clear(); }
const char* t_elsewhere() { return g_elsewhere.c_str(); }
int t_allocs() { return g_allocs; }
void t_set_device(int device) { g_device = device; }

hipError_t hipGetDeviceCount(int* n) { *n = 2; return hipSuccess; }
hipError_t hipSetDevice(int d) { g_device = d; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipMalloc(void** p, size_t n) { ++g_allocs; *p = calloc(1, n ? n : 1); return (hipError_t)work("hipMalloc"); }
hipError_t hipFree(void* p) { ++g_allocs; free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n ? n : 1); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    memcpy(d, s, n);
    return (hipError_t)work("hipMemcpyAsync");
}
hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return (hipError_t)work("hipMemset"); }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)malloc(1); return (hipError_t)work("hipEventCreate"); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free((void*)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)malloc(1); return (hipError_t)work("hipStreamCreate"); }
hipError_t hipStreamDestroy(hipStream_t s) { free((void*)s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}

namespace mvf {
int launch_frame_prep(const PrepItem*, int, int, int, void*, const void*, void*, size_t) { return work("frame_prep"); }
int launch_volume_init(DevVolume, void*) { return work("volume_init"); }
int launch_ztable(const IntegrateLaunch&, int, void*) { return work("ztable"); }
int launch_integrate(const IntegrateLaunch&, int, void*, void*, void*) { return work("integrate"); }
int launch_raycast(const RaycastLaunch&, int, void*, void*, void*) { return work("raycast"); }
int launch_column_flags(DevVolume, void*) { return work("column_flags"); }
int launch_brick_distance(const LaunchHeader*, const DevVolume*, const int32_t*, int, int, void*, const DevFrame*,
                          RayBounds) { return work("brick_distance"); }
int launch_ray_bounds_collect(const LaunchHeader*, const DevVolume*, const int32_t*, const DevFrame*, RayBounds, int,
                              void*) { return work("ray_bounds_collect"); }
int launch_ray_bounds_merge(const LaunchHeader*, const DevFrame*, const int32_t*, const int32_t*, const int32_t*,
                            RayBounds, int, int, int, void*, TileOrder) { return work("ray_bounds_merge"); }
int launch_swap_copy(const void* src, void* dst, size_t bytes, void*)
{
    memcpy(dst, src, bytes);
    return work("swap_copy");
}
int launch_read_plane(DevVolume, int plane, uint32_t, uint32_t n, void* out, void*)
{
    memset(out, 0, (size_t)n * (plane == 1 ? 2 : 4));
    return work("read_plane");
}
int launch_import(DevVolume, const float*, const uint16_t*, const uint32_t*, bool, void*) { return work("import"); }
size_t extract_buffer_bytes(size_t nbricks) { return 64 * nbricks; }
ExtractBuffers extract_buffers(void*, size_t, long long* total)
{
    ExtractBuffers B{};
    B.total = total;
    return B;
}
int launch_extract(DevVolume, const ExtractBuffers&, float*, float*, int32_t*, long long, void*) { return work("extract"); }
int launch_placement_clear(unsigned long long*, int, int*, void*) { return work("placement_clear"); }
int launch_placement_count(const PlacementCount&, PlacementCells* out, void*)
{
    out->n = out->overflow = 0;
    return work("placement_count");
}
int launch_track_smooth(const float*, int, int, int, float, float*, void*) { return work("track_smooth"); }
int launch_track_down(const float*, int, int, int, float, float*, void*) { return work("track_down"); }
int launch_track_maps(TrackMaps, void*) { return work("track_maps"); }
int track_blocks(int, int) { return 1; }
int launch_icp_step(const TrackLaunch&, int, TrackState*, void*) { return work("icp_step"); }
int diffray_scratch_init(int) { return 0; }
double* diffray_scratch(int) { return nullptr; }
int diffray_partials_needed(int, int) { return 1; }
int launch_diffray_backward(DiffVolume, const float*, float, float, float, float, int, int, RayParams, const float*,
                            const int32_t*, float*, double*, int, double*, void*) { return work("diffray_backward"); }
}  // namespace mvf
