// A HIP runtime that runs nothing and records what the library asks of it:
// every launch (device, kernel, grid, block, dynamic LDS) with the dynamic-LDS
// limit that had been set for that kernel on that device.  Loaded ahead of
// libsd.so, whose calls then bind to it; no GPU is needed.
#include <cstddef>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

namespace {
struct Dim { unsigned x, y, z; };
struct Launch { int dev; std::string name; Dim grid, block; size_t lds; int limit; };
struct Config { Dim grid, block; size_t lds; void* stream; };
std::mutex mu;
std::map<const void*, std::string> names;
std::map<std::pair<int, const void*>, int> limits;
std::vector<Launch> launches;
int device = 0;
thread_local std::vector<Config> configs;
alignas(256) unsigned char symbol[256];

int record(const void* f, Dim grid, Dim block, size_t lds) {
  std::lock_guard<std::mutex> l(mu);
  auto it = limits.find({device, f});
  launches.push_back({device, names[f], grid, block, lds, it == limits.end() ? 0 : it->second});
  return 0;
}
}  // namespace

extern "C" {
void recorder_device(int d) { device = d; }
void recorder_clear() { launches.clear(); }
int recorder_count() { return (int)launches.size(); }
void recorder_get(int i, char* name, int cap, int* v) {
  const Launch& l = launches[i];
  snprintf(name, cap, "%s", l.name.c_str());
  const int w[] = {l.dev, (int)(l.grid.x * l.grid.y * l.grid.z), (int)l.block.x, (int)l.lds, l.limit};
  memcpy(v, w, sizeof(w));
}

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, Dim*, Dim*, int*) {
  names[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim g, Dim b, size_t lds, void* s) { configs.push_back({g, b, lds, s}); return 0; }
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* lds, void** s) {
  const Config c = configs.back();
  configs.pop_back();
  *g = c.grid; *b = c.block; *lds = c.lds; *s = c.stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim g, Dim b, void**, size_t lds, void*) { return record(f, g, b, lds); }
int hipExtLaunchKernel(const void* f, Dim g, Dim b, void**, size_t lds, void*, void*, void*, int) { return record(f, g, b, lds); }
int hipFuncSetAttribute(const void* f, int attr, int value) {
  std::lock_guard<std::mutex> l(mu);
  if (attr == 8) limits[{device, f}] = value;   // hipFuncAttributeMaxDynamicSharedMemorySize
  return 0;
}
int hipGetDevice(int* d) { *d = device; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = symbol; return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return ""; }
int hipMemcpy(void*, const void*, size_t, int) { return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipEventCreate(void** e) { *e = symbol; return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 0.f; return 0; }
}
