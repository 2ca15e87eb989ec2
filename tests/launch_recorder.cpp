// Host runtime without a GPU: the HIP calls and kernel launches that
// runtime.cpp, server.cpp and static_rollout.cpp make, as stubs that allocate
// host memory and record what would have been launched.  Built by
// test_launch_routes.py together with those files.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <vector>

#include "launch.h"
#include "render.h"

namespace {

enum : int32_t { kPlain = 0, kFused = 1, kReset = 2 };

struct Launch {
  int32_t kind, tile_envs, n_tiles, blocks, max_cells, steps, balls, corridors;
};

std::vector<Launch> launches;

}  // namespace

extern "C" {

int32_t rec_take(Launch* out, int32_t cap) {
  const int32_t n = (int32_t)launches.size();
  for (int32_t i = 0; i < n && i < cap; ++i) out[i] = launches[i];
  launches.clear();
  return n;
}

hipError_t hipMalloc(void** p, size_t n) {
  *p = calloc(1, n ? n : 1);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) {
  return hipMemcpy(d, s, n, k);
}
hipError_t hipMemset(void* d, int v, size_t n) {
  memset(d, v, n);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned) { return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  static int event;
  *e = reinterpret_cast<hipEvent_t>(&event);
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) {
  *p = const_cast<void*>(s);
  return hipSuccess;
}

}  // extern "C"

namespace gx {

hipError_t launch_plain(const EnvTables&, const StateBufs&, const uint8_t*, const TrajBufs&, int32_t, bool balls,
                        hipStream_t) {
  launches.push_back({kPlain, 0, 0, 0, 0, 1, balls, 0});
  return hipSuccess;
}

hipError_t launch_reset(const EnvTables&, const TileTables& t, const StateBufs&, const TrajBufs&, hipStream_t) {
  launches.push_back({kReset, t.tile_envs, t.n_tiles, t.n_tiles, t.max_tile_cells, 0, 0, t.corridors});
  return hipSuccess;
}

hipError_t launch_fused(const EnvTables&, const TileTables& t, const StateBufs&, const uint8_t*, int32_t k_steps,
                        const TrajBufs&, int32_t, int32_t blocks, hipStream_t, ServeTile*, const ServeTile*,
                        const SlotConfig*) {
  launches.push_back({kFused, t.tile_envs, t.n_tiles, blocks, t.max_tile_cells, k_steps, 0, t.corridors});
  return hipSuccess;
}

size_t fused_dynamic_lds_bytes(int32_t cells) { return (size_t)cells + 384; }
size_t fused_lds_bytes(int32_t cells, bool pairs) { return (size_t)cells + (pairs ? 1 : 0); }

hipError_t launch_render(const RenderSrc&, int32_t, int32_t, bool, const uint2*, uint32_t, const uint8_t*,
                         const RenderDst&, int32_t, hipStream_t) {
  return hipSuccess;
}

}  // namespace gx
