// Host check (no GPU): after clue_create, runs and read-outs allocate nothing, the
// first ones included. The HIP calls of the host runtime are answered here, out of
// host memory, and those that allocate are counted.
#include "clue_api.hip"

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
static hipError_t ran(const Arena& a, const RunDesc& d) {
  if (a.fstart) a.fstart[d.n] = kFollowers;
  return hipSuccess;
}
hipError_t launch_pipeline(const Geom&, const Arena& a, const RunDesc& d, const LaunchCfg&, hipStream_t, hipEvent_t*) {
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

int main() {
  constexpr int N = 20000;
  std::vector<float> f(N), rho(N), d2(N);
  std::vector<int32_t> i(N), nh(N), cid(N), fstart(N + 1), flist(N);
  std::vector<uint8_t> seed(N);
  clue_params p{};
  p.dc = 2.0f;
  p.delta_c = 2.0f;
  p.delta_o = 4.0f;
  p.x_max = p.y_max = 50.0f;
  p.n_layers = 3;
  p.flags = CLUE_KEEP_INTERMEDIATES;
  for (int n : {100, N}) {  // the all-pairs and the tiled form
    for (int batched = 0; batched < 2; ++batched) {
      clue_ctx* c = nullptr;
      if (clue_create(&c, &p, 0, N, 2, 0) != CLUE_OK) {
        std::printf("clue_create: %s\n", clue_last_error(nullptr));
        return 1;
      }
      const int created = g_allocations;
      int64_t total = -1;
      const int rc[] = {
          batched ? clue_run_batch(c, n, 2, i.data(), f.data(), f.data(), i.data(), f.data(), cid.data(), seed.data(), nullptr)
                  : clue_run(c, n, f.data(), f.data(), i.data(), f.data(), cid.data(), seed.data(), nullptr),
          clue_get_intermediates(c, rho.data(), nh.data(), d2.data(), nullptr),
          clue_get_followers(c, fstart.data(), flist.data(), nullptr, nullptr),
          clue_get_followers(c, fstart.data(), flist.data(), &total, nullptr),
      };
      const char* const what[] = {"the run", "clue_get_intermediates", "clue_get_followers", "clue_get_followers with its number"};
      for (int k = 0; k < 4; ++k)
        if (rc[k] != CLUE_OK) {
          std::printf("%s: %s\n", what[k], clue_last_error(c));
          return 1;
        }
      if (total != kFollowers) {
        std::printf("%lld followers, want %d\n", (long long)total, kFollowers);
        return 1;
      }
      if (g_allocations != created) {
        std::printf("%d hits, batched %d: %d allocations after clue_create\n", n, batched, g_allocations - created);
        return 1;
      }
      clue_destroy(c);
    }
  }
  std::printf("none\n");
  return 0;
}
