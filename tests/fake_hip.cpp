// The few HIP entry points that libpctree.so imports, without a device: loaded
// ahead of it, they record every kernel launch (name, grid, block, dynamic LDS) and
// can be told to fail.  A host-side check of what a call would launch.
#include <hip/hip_runtime_api.h>

#include <map>
#include <string>
#include <vector>

namespace {
struct Launch {
  std::string name;
  dim3 grid, block;
  size_t lds;
};
std::map<const void*, std::string> g_names;
std::vector<Launch> g_launches;
Launch g_config;
hipError_t g_last = hipSuccess;
int g_fail_attributes = 0, g_fail_occupancy = 0, g_cus = 256;

hipError_t result(int& failures) {
  if (failures <= 0) return hipSuccess;
  --failures;
  return g_last = hipErrorUnknown;
}
}  // namespace

extern "C" {

void fake_reset(int cus, int fail_attributes, int fail_occupancy) {
  g_launches.clear();
  g_cus = cus;
  g_fail_attributes = fail_attributes;
  g_fail_occupancy = fail_occupancy;
}
int fake_launches() { return (int)g_launches.size(); }
const char* fake_launch(int i, unsigned* grid, unsigned* block, size_t* lds) {
  const Launch& l = g_launches[i];
  *grid = l.grid.x;
  *block = l.block.x;
  *lds = l.lds;
  return l.name.c_str();
}

void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
  g_names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t) {
  g_config = {"", grid, block, lds};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* st) {
  *grid = g_config.grid;
  *block = g_config.block;
  *lds = g_config.lds;
  *st = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3 grid, dim3 block, void**, size_t lds, hipStream_t) {
  g_launches.push_back({g_names[fn], grid, block, lds});
  return hipSuccess;
}
hipError_t hipGetDevice(int* dev) {
  *dev = 0;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  const hipError_t e = result(g_fail_attributes);
  if (e != hipSuccess) return e;
  *v = a == hipDeviceAttributeMultiprocessorCount         ? g_cus
       : a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 160 * 1024
                                                         : 100000;
  return hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes* attr, const void*) {
  *attr = hipFuncAttributes{};
  attr->sharedSizeBytes = 12 * 1024;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 1;
  return result(g_fail_occupancy);
}
hipError_t hipGetSymbolAddress(void** ptr, const void*) {
  *ptr = (void*)0x10000000;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = (hipEvent_t)0x1;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.0f;
  return hipSuccess;
}

}  // extern "C"
