// A HIP runtime of one device with a given amount of memory, for the host side of the
// library on a machine without a GPU: preloaded, it takes the place of the calls that
// creating and destroying a handle makes.  Device addresses are never followed.  With
// FAKE_HIP_DRIVER it is a program instead: it creates a handle (arguments: n_envs,
// ckpt_every, max_tape_horizon) and prints the status and every allocation.
#ifndef FAKE_HIP_DRIVER
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

static size_t total() {
  const char* s = std::getenv("FAKE_HIP_BYTES");
  return s ? std::strtoull(s, nullptr, 10) : (size_t)1 << 40;
}
static size_t used = 0;
static uintptr_t next_address = 1 << 20;
static std::map<void*, size_t>& sizes() {
  static std::map<void*, size_t> m;
  return m;
}

extern "C" {
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
  if (n > total() - used) return hipErrorOutOfMemory;
  *p = reinterpret_cast<void*>(next_address);
  next_address += (n + 255) & ~(size_t)255;
  used += n;
  sizes()[*p] = n;
  std::printf("malloc %zu\n", n);
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  used -= sizes()[p];
  sizes().erase(p);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* free_bytes, size_t* all) {
  const char* s = std::getenv("FAKE_HIP_FREE");  // what is reported, not what there is
  *free_bytes = s ? std::strtoull(s, nullptr, 10) : total() - used;
  *all = total();
  return hipSuccess;
}
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = reinterpret_cast<void*>(4096); return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipPeekAtLastError() { return hipSuccess; }
}
#else
#include <dlfcn.h>

#include <cstdio>
#include <cstdlib>

#include "quadsim.h"

int main(int argc, char** argv) {
  void* lib = dlopen(argv[1], RTLD_NOW);
  if (!lib) {
    std::printf("dlopen %s\n", dlerror());
    return 2;
  }
  auto create = reinterpret_cast<decltype(&sim_create)>(dlsym(lib, "sim_create"));
  auto destroy = reinterpret_cast<decltype(&sim_destroy)>(dlsym(lib, "sim_destroy"));
  sim_config c{};
  c.n_envs = std::atoi(argv[2]);
  c.ckpt_every = std::atoi(argv[3]);
  c.max_tape_horizon = std::atoi(argv[4]);
  c.flags = SIM_F_RENORM_Q;
  c.dt = 0.01, c.g = 9.81, c.arm = 0.028, c.k_m = 6e-3, c.rpm_max = 21702.0;
  const double nominal[8] = {0.027, 3.85e-6, 3.85e-6, 5.9675e-6, 0, 0, 3.16e-10, 0.15};
  for (int i = 0; i < 8; ++i) c.nominal[i] = nominal[i], c.dr_lo[i] = c.dr_hi[i] = 1.0;
  c.pos_limit = c.vel_limit = 1.0;
  sim_handle* h = nullptr;
  const int rc = create(&c, 0, &h);
  std::printf("rc %d\n", rc);
  if (h) destroy(h);
  return 0;
}
#endif
