// A host-only stand-in for the HIP runtime calls that libwfs.so makes, so that what the library
// decides on the host (which sizes it takes, what it launches, allocates and clears, and when)
// can be checked without a GPU.  Device memory is host memory, kernels are not run but written
// down, and a launch with more than 64 KB of dynamic LDS is refused unless the kernel was
// allowed that much on the current device.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <utility>

struct Dim3 {
  uint32_t x, y, z;
};

static int g_device = 0, g_capturing = 0, g_refuse_attr = 0, g_error = 0;
static int g_fail_launch = -1;  // launches until one fails (-1: none does)
static uint64_t g_handles = 0;
static std::map<const void*, std::string> g_names;
static std::map<std::pair<int, const void*>, int> g_lds;  // (device, kernel): bytes allowed
static std::string g_log;
static Dim3 g_grid, g_block;
static size_t g_shm;
static void* g_stream;
static char g_symbol[64];

static void log_line(const char* what, const void* kernel, long long a, long long b) {
  char buf[512];
  const auto it = g_names.find(kernel);
  snprintf(buf, sizeof buf, "%s %s %lld %lld\n", what, it == g_names.end() ? "-" : it->second.c_str(),
           a, b);
  g_log += buf;
}

extern "C" {

// Test side: the current device, whether streams are capturing, whether attributes are refused,
// the launch that fails (counted from 0; -1: none), and the lines written since the last call
// ("launch name blocks lds" / "malloc - bytes 0" / "attr name device bytes", and the order of
// streams: "on - stream 0" for a launch, "record - stream event", "wait - stream event").
void rec_set(int device, int capturing, int refuse_attr) {
  g_device = device;
  g_capturing = capturing;
  g_refuse_attr = refuse_attr;
}
void rec_fail_launch(int n) { g_fail_launch = n; }
const char* rec_take() {
  static std::string out;
  out.swap(g_log);
  g_log.clear();
  return out.c_str();
}

void** __hipRegisterFatBinary(const void*) { return reinterpret_cast<void**>(&g_handles); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  g_names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shm, void* stream) {
  g_grid = grid;
  g_block = block;
  g_shm = shm;
  g_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shm, void** stream) {
  *grid = g_grid;
  *block = g_block;
  *shm = g_shm;
  *stream = g_stream;
  return 0;
}
int hipLaunchKernel(const void* kernel, Dim3 grid, Dim3, void**, size_t shm, void* stream) {
  if (g_fail_launch >= 0 && g_fail_launch-- == 0) return g_error = 1;
  log_line("on", nullptr, (long long)stream, 0);
  const auto it = g_lds.find({g_device, kernel});
  log_line("launch", kernel, (long long)grid.x * grid.y * grid.z, (long long)shm);
  if (shm > 65536 && (it == g_lds.end() || (size_t)it->second < shm)) {
    log_line("refused", kernel, g_device, (long long)shm);
    g_error = 1;
  }
  return g_error;
}
int hipFuncSetAttribute(const void* kernel, int, int value) {
  log_line("attr", kernel, g_device, value);
  if (g_refuse_attr) return 1;
  g_lds[{g_device, kernel}] = value;
  return 0;
}
int hipGetDevice(int* d) {
  *d = g_device;
  return 0;
}
int hipDeviceGetAttribute(int* v, int, int) {
  *v = 256;
  return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 2;
  return 0;
}
int hipMalloc(void** p, size_t n) {
  log_line("malloc", nullptr, (long long)n, 0);
  *p = malloc(n ? n : 1);
  return *p ? 0 : 2;
}
int hipFree(void* p) {
  free(p);
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
  memcpy(d, s, n);
  return 0;
}
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipMemset(void* d, int v, size_t n) {
  memset(d, v, n);
  return 0;
}
int hipDeviceSynchronize() { return 0; }
const char* hipGetErrorString(int) { return "recorded error"; }
int hipGetLastError() {
  const int e = g_error;
  g_error = 0;
  return e;
}
int hipGetSymbolAddress(void** p, const void*) {
  *p = g_symbol;
  return 0;
}
int hipEventCreate(void** e) {
  *e = reinterpret_cast<void*>(++g_handles);
  return 0;
}
int hipEventCreateWithFlags(void** e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void* event, void* stream) {
  log_line("record", nullptr, (long long)stream, (long long)event);
  return 0;
}
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) {
  *ms = 1.0f;
  return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned) { return hipEventCreate(s); }
int hipStreamDestroy(void*) { return 0; }
int hipStreamIsCapturing(void*, int* status) {
  *status = g_capturing;
  return 0;
}
int hipStreamWaitEvent(void* stream, void* event, unsigned) {
  log_line("wait", nullptr, (long long)stream, (long long)event);
  return 0;
}

}  // extern "C"
