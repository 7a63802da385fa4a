// Stands in for the HIP runtime in front of the library's host code, on a machine without a GPU: two devices, no kernels.  What
// is enqueued is written down in order, a word per call; recorder_log returns it.  Loaded with global symbols before the
// library, whose calls then end here.
#include <cstddef>
#include <cstdio>
#include <string>

namespace {
std::string g_log;
int g_device = 0, g_mode = 0;             // capture mode of the thread: 0 global, 2 relaxed
long g_events = 0;
void note(const char* what, const void* a = nullptr, const void* b = nullptr) {
    char line[96];
    std::snprintf(line, sizeof line, "%s %zu %zu\n", what, reinterpret_cast<size_t>(a), reinterpret_cast<size_t>(b));
    g_log += line;
}
}  // namespace

extern "C" {
const char* recorder_log() { return g_log.c_str(); }
void recorder_clear() { g_log.clear(); }

int hipGetDeviceCount(int* n) { *n = 2; return 0; }
int hipGetDevice(int* d) { *d = g_device; return 0; }
int hipSetDevice(int d) { g_device = d; return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "recorded"; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = reinterpret_cast<void*>(0x1000 + 16 * ++g_events); return 0; }
int hipEventCreate(void** e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void* e, void* stream) {
    note(stream ? "record" : g_device ? "record-elsewhere" : g_mode == 2 ? "record-relaxed" : "record", e, stream);
    return 0;
}
int hipStreamWaitEvent(void* stream, void* e, unsigned) { note("wait", stream, e); return 0; }
int hipStreamIsCapturing(void*, int* status) { *status = 0; return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipThreadExchangeStreamCaptureMode(int* mode) { const int old = g_mode; g_mode = *mode; *mode = old; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = reinterpret_cast<void*>(0x10000); return 0; }
struct Dim3 { unsigned x, y, z; };
static struct { Dim3 grid, block; size_t lds; void* stream; } g_launch;
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) { g_launch = {grid, block, lds, stream}; return 0; }
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
    *grid = g_launch.grid; *block = g_launch.block; *lds = g_launch.lds; *stream = g_launch.stream;
    return 0;
}
int hipLaunchKernel(const void*, Dim3, Dim3, void**, size_t, void* stream) { note("launch", stream, reinterpret_cast<void*>((size_t)g_device)); return 0; }
}
