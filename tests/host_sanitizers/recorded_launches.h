// A HIP runtime for the host checks that launches nothing: the definitions here take the place of the runtime's own in the
// executable they are linked into.  Launches and LDS opt-ins are recorded, devices are numbers.
#pragma once
#include <hip/hip_runtime.h>
#include <string.h>

#include <map>
#include <utility>
#include <vector>

struct RecordedLaunch {
  const void* kernel;
  dim3 grid, block;
  size_t lds;
  int device, lds_allowed;             // dynamic LDS the kernel was opted in for on that device (64 KiB where it was not)
  std::vector<int> ints;               // the arguments listed in g_record_ints
};
static std::vector<RecordedLaunch> g_launches;
static std::map<std::pair<int, const void*>, int> g_opted_in;
static int g_device = 0;
static std::vector<int> g_record_ints;   // indexes of kernel arguments that are ints

extern "C" hipError_t hipGetDevice(int* d) { *d = g_device; return hipSuccess; }
extern "C" hipError_t hipSetDevice(int d) { g_device = d; return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
extern "C" hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
extern "C" hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 2; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int v) {
  g_opted_in[{g_device, f}] = v;
  return hipSuccess;
}
// <<<grid, block, lds, stream>>> leaves the configuration for the kernel's host stub, which fetches it and calls hipLaunchKernel
static struct { dim3 grid, block; size_t lds; hipStream_t stream; } g_config;
extern "C" hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  g_config = {grid, block, lds, stream};
  return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  *grid = g_config.grid;
  *block = g_config.block;
  *lds = g_config.lds;
  *stream = g_config.stream;
  return hipSuccess;
}
extern "C" hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t) {
  RecordedLaunch l{f, grid, block, lds, g_device, 64 * 1024, {}};
  const auto it = g_opted_in.find({g_device, f});
  if (it != g_opted_in.end()) l.lds_allowed = it->second;
  for (int i : g_record_ints) {
    int v;
    memcpy(&v, args[i], sizeof v);
    l.ints.push_back(v);
  }
  g_launches.push_back(l);
  return hipSuccess;
}
