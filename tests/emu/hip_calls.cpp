// hip_calls.cpp -- stand-ins for the HIP runtime calls of libfvm.so's host code,
// preloaded in front of the runtime so that a test without a GPU sees what the
// library asks for: every launch, event record and wait is a line of a log.
// Nothing runs. A stream handle names its device (bits 16 and up); the null
// stream is the current device's.
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <string>
#include <utility>
#include <vector>

namespace {
std::string g_log;
int g_device = 0;
std::vector<int> g_event_device;
std::vector<bool> g_event_over;  // what was recorded last is over (see calls_finish)
struct Config {
  unsigned grid[3], block[3];
  size_t shared;
  void* stream;
} g_config;
int device_of(void* stream) {
  return stream ? static_cast<int>(reinterpret_cast<uintptr_t>(stream) >> 16) : g_device;
}
void note(const char* what, uintptr_t a, uintptr_t b, uintptr_t c) {
  char line[128];
  std::snprintf(line, sizeof line, "%s %zu %zu %zu\n", what, static_cast<size_t>(a),
                static_cast<size_t>(b), static_cast<size_t>(c));
  g_log += line;
}
}  // namespace

struct dim3 {
  uint32_t x, y, z;
};
struct NodeParams {  // hipKernelNodeParams
  dim3 block;
  void** extra;
  void* func;
  dim3 grid;
};

extern "C" {

// for the test
const char* calls_log() { return g_log.c_str(); }
void calls_clear() { g_log.clear(); }
void calls_device(int device) { g_device = device; }
void calls_finish() { g_event_over.assign(g_event_over.size(), true); }  // the GPU is idle

int hipGetDevice(int* d) {
  *d = g_device;
  return 0;
}
int hipDeviceGetAttribute(int* v, int, int) {
  *v = 256;  // compute units
  return 0;
}
int hipStreamGetDevice(void* s, int* d) {
  *d = device_of(s);
  return 0;
}
int hipStreamIsCapturing(void*, int* status) {
  *status = 0;
  return 0;
}
int hipStreamSynchronize(void*) { return 0; }
int hipGetLastError() { return 0; }
int hipMemcpy(void*, const void*, size_t, int) { return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }

// events are 1, 2, ..; recording one on another device's stream fails
int hipEventCreateWithFlags(void** e, unsigned) {
  g_event_device.push_back(g_device);
  g_event_over.push_back(true);
  *e = reinterpret_cast<void*>(g_event_device.size());
  return 0;
}
int hipEventRecord(void* e, void* s) {
  const uintptr_t k = reinterpret_cast<uintptr_t>(e);
  if (k == 0 || k > g_event_device.size() || g_event_device[k - 1] != device_of(s)) return 400;
  g_event_over[k - 1] = false;
  note("record", k, reinterpret_cast<uintptr_t>(s), 0);
  return 0;
}
int hipEventQuery(void* e) {
  return g_event_over[reinterpret_cast<uintptr_t>(e) - 1] ? 0 : 600;
}
int hipThreadExchangeStreamCaptureMode(int* mode) {
  static int now = 0;
  std::swap(*mode, now);
  return 0;
}
int hipStreamWaitEvent(void* s, void* e, unsigned) {
  note("wait", reinterpret_cast<uintptr_t>(e), reinterpret_cast<uintptr_t>(s), 0);
  return 0;
}

int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void* stream) {
  g_config = {{grid.x, grid.y, grid.z}, {block.x, block.y, block.z}, shared, stream};
  return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, void** stream) {
  *grid = {g_config.grid[0], g_config.grid[1], g_config.grid[2]};
  *block = {g_config.block[0], g_config.block[1], g_config.block[2]};
  *shared = g_config.shared;
  *stream = g_config.stream;
  return 0;
}
int hipLaunchKernel(const void*, dim3 grid, dim3 block, void**, size_t, void* stream) {
  note("launch", grid.x, block.x, reinterpret_cast<uintptr_t>(stream));
  return 0;
}

int hipGraphCreate(void** g, unsigned) {
  *g = reinterpret_cast<void*>(1);
  return 0;
}
int hipGraphAddKernelNode(void** n, void*, void**, size_t, NodeParams*) {
  *n = reinterpret_cast<void*>(1);
  return 0;
}
int hipGraphInstantiate(void** e, void*, void**, char*, size_t) {
  *e = reinterpret_cast<void*>(1);
  return 0;
}
int hipGraphLaunch(void*, void* stream) {
  note("graph", 0, 0, reinterpret_cast<uintptr_t>(stream));
  return 0;
}
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }

}  // extern "C"
