// A HIP runtime of the calls that libburgers.so makes, for tests of its host code without a GPU: memory is host
// memory, kernels do nothing, and streams, events and launches are counted.  Loaded ahead of libburgers.so under the
// runtime's soname.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <set>

extern "C" {

struct dim { uint32_t x, y, z; };
typedef void* handle;

static long streams_made, streams_live, events_made, events_live, launches, copies;
static std::set<handle>* used;   // streams that launches went to

void fake_reset() {
  streams_made = events_made = launches = copies = 0;
  if (used) used->clear();
}
long fake_streams_made() { return streams_made; }
long fake_streams_live() { return streams_live; }
long fake_events_made() { return events_made; }
long fake_events_live() { return events_live; }
long fake_launches() { return launches; }
long fake_streams_used() { return used ? static_cast<long>(used->size()) : 0; }
int fake_stream_used(handle s) { return used && used->count(s) ? 1 : 0; }

int hipStreamCreateWithFlags(handle* s, unsigned) { ++streams_made; ++streams_live; *s = malloc(1); return 0; }
int hipStreamDestroy(handle s) { --streams_live; free(s); return 0; }
int hipStreamSynchronize(handle) { return 0; }
int hipStreamWaitEvent(handle, handle, unsigned) { return 0; }
int hipStreamBeginCapture(handle, int) { return 0; }
int hipStreamEndCapture(handle, handle* g) { *g = malloc(1); return 0; }
int hipGraphInstantiate(handle* e, handle, handle*, char*, size_t) { *e = malloc(1); return 0; }
int hipGraphLaunch(handle, handle) { return 0; }
int hipGraphDestroy(handle g) { free(g); return 0; }
int hipGraphExecDestroy(handle g) { free(g); return 0; }
int hipEventCreateWithFlags(handle* e, unsigned) { ++events_made; ++events_live; *e = malloc(1); return 0; }
int hipEventCreate(handle* e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(handle e) { --events_live; free(e); return 0; }
int hipEventRecord(handle, handle) { return 0; }
int hipEventQuery(handle) { return 0; }
int hipEventSynchronize(handle) { return 0; }
int hipEventElapsedTime(float* ms, handle, handle) { *ms = 1.0f; return 0; }
int hipMallocAsync(void** p, size_t n, handle) { *p = malloc(n); return *p ? 0 : 2; }
int hipFreeAsync(void* p, handle) { free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = malloc(n); return *p ? 0 : 2; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, handle) { ++copies; memmove(d, s, n); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { memmove(d, s, n); return 0; }
int hipMemsetAsync(void* d, int v, size_t n, handle) { memset(d, v, n); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 1; return 0; }
int hipGetSymbolAddress(void** p, const void*) {
  static void* scratch = malloc(size_t{64} << 20);
  *p = scratch;
  return 0;
}
int hipLaunchKernel(const void*, dim, dim, void**, size_t, handle s) {
  ++launches;
  if (!used) used = new std::set<handle>;
  used->insert(s);
  return 0;
}
static thread_local struct { dim grid, block; size_t shared; handle stream; } call;
int __hipPushCallConfiguration(dim g, dim b, size_t n, handle s) { call = {g, b, n, s}; return 0; }
int __hipPopCallConfiguration(dim* g, dim* b, size_t* n, handle* s) {
  *g = call.grid; *b = call.block; *n = call.shared; *s = call.stream;
  return 0;
}
void** __hipRegisterFatBinary(const void*) { static void* none; return &none; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

}  // extern "C"
