// The HIP calls that the host runtime makes in a context's life and its runs,
// answered out of host memory, and the kernels' side of the library. Included after
// clue_api.hip by programs that check the host runtime without a GPU.
#pragma once

static int g_allocations = 0;

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { return ++g_allocations, *p = std::calloc(1, n), hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return ++g_allocations, *p = std::calloc(1, n), hipSuccess; }
hipError_t hipFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipHostFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) { return p->multiProcessorCount = 256, hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = nullptr, hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }  // calloc's
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) {
  a->type = hipMemoryTypeDevice;
  a->device = 0;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
  *base = p;
  *size = (size_t)1 << 40;
  return hipSuccess;
}
}  // extern "C"

namespace clue {
const char* const kStageNames[S_COUNT] = {};
constexpr int kFollowers = 37;  // of every run
static Geom g_ran{};            // the geometry of the last tiled run
static bool g_graph = false;    // and whether the context's graph was captured for it
static hipError_t ran(const Arena& a, const RunDesc& d) {
  if (a.fstart) a.fstart[d.n] = kFollowers;
  return hipSuccess;
}
hipError_t launch_pipeline(const Geom& g, const Arena& a, const RunDesc& d, const LaunchCfg& cfg, hipStream_t, hipEvent_t*) {
  g_ran = g;
  g_graph = cfg.graph_mode;
  return ran(a, d);
}
hipError_t launch_direct(const Geom&, const Arena& a, const RunDesc& d, hipStream_t, hipEvent_t*) { return ran(a, d); }
hipError_t launch_set_desc(const RunDesc&, RunDesc*, hipStream_t) { return hipSuccess; }
hipError_t launch_read_out(const ReadOut& r, hipStream_t) {
  for (int k = 0; k < 3; ++k)
    if (r.dst[k]) std::memcpy(r.dst[k], r.src[k], (size_t)r.n[k] * 4);
  if (r.word_out) *r.word_out = *r.word;
  return hipSuccess;
}
hipError_t launch_event_ids(int32_t*, const int64_t*, int32_t, int32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_validate(const Geom&, const Arena&, const RunDesc&, hipStream_t) { return hipSuccess; }
int occupancy_blocks_per_cu(int, int) { return 1; }
int lds_bytes_for(const Geom&) { return 0; }
int lds_bytes_nh(const Geom&) { return 0; }
}  // namespace clue
