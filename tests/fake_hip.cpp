// The part of the HIP runtime that libgw.so calls, on host memory and with nothing launched, so that the library's
// host side (workspace, copies, the choice of kernels, what a stream capture records) can be tested without a GPU.
// Loaded before the library with RTLD_GLOBAL, its symbols take the runtime's place.
//
// Device memory is host memory; a freed block is handed out again, with its contents, to the next request of its
// size.  Copies run at once, or are recorded while their stream captures; fake_replay() runs the recorded ones.
// Allocating, freeing or synchronising during a capture fails, as the runtime does, and is counted.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

struct dim3 { uint32_t x, y, z; };
typedef void *stream_t;
enum { OK = 0, OUT_OF_MEMORY = 2, CAPTURE_UNSUPPORTED = 900 };

namespace {
struct Copy { void *dst; const void *src; size_t bytes; };
struct Launch { std::string name; dim3 grid, block; bool captured; };
std::map<const void *, std::string> names;
std::map<void *, size_t> blocks;
std::map<size_t, std::vector<void *>> freed;
std::map<stream_t, bool> capturing;
std::vector<Copy> recorded;
std::vector<Launch> launches;
size_t limit = 0;                       // requests above it fail (0: none do)
float cut_ms = 1.0f;                    // time between two events after a launch that adds parts of cut tiles
int last = OK, violations = 0, copies = 0, mallocs = 0;
struct Config { dim3 grid, block; size_t shared; stream_t s; } config;

bool any_capture() {
  for (auto &c : capturing)
    if (c.second) return true;
  return false;
}
int fail(int e) { return last = e; }
int in_capture() {
  ++violations;
  return fail(CAPTURE_UNSUPPORTED);
}
}  // namespace

extern "C" {

// ---- for the test --------------------------------------------------------------------------------------
void fake_limit(size_t bytes) { limit = bytes; }
void fake_cut_ms(float ms) { cut_ms = ms; }
void fake_capture(stream_t s, int on) { capturing[s] = on != 0; }
int fake_violations() { return violations; }
int fake_recorded() { return (int)recorded.size(); }
const void *fake_recorded_src(int i) { return recorded[(size_t)i].src; }
size_t fake_recorded_bytes(int i) { return recorded[(size_t)i].bytes; }
void *fake_recorded_dst(int i) { return recorded[(size_t)i].dst; }
void fake_replay() {
  for (const Copy &c : recorded) memcpy(c.dst, c.src, c.bytes);
}
int fake_copies() { return copies; }
int fake_mallocs() { return mallocs; }          // requests, those that failed among them
int fake_launches() { return (int)launches.size(); }
const char *fake_launch_name(int i) { return launches[(size_t)i].name.c_str(); }
unsigned fake_launch_grid(int i) { return launches[(size_t)i].grid.x; }
int fake_launch_captured(int i) { return launches[(size_t)i].captured; }
void fake_clear() {
  launches.clear();
  recorded.clear();
  copies = 0;
}
int fake_is_block(const void *p) {      // inside a live allocation
  for (auto &b : blocks)
    if (p >= b.first && p < (char *)b.first + b.second) return 1;
  return 0;
}

// ---- the runtime -----------------------------------------------------------------------------------------
void **__hipRegisterFatBinary(const void *) {
  static void *handle;
  return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *,
                           void *, int *) {
  names[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, stream_t s) {
  config = {grid, block, shared, s};
  return OK;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, stream_t *s) {
  *grid = config.grid;
  *block = config.block;
  *shared = config.shared;
  *s = config.s;
  return OK;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **, size_t, stream_t s) {
  auto n = names.find(f);
  launches.push_back({n == names.end() ? "?" : n->second, grid, block, capturing[s]});
  return OK;
}
int hipMalloc(void **p, size_t bytes) {
  ++mallocs;
  if (any_capture()) return in_capture();
  if (limit && bytes > limit) return fail(OUT_OF_MEMORY);
  std::vector<void *> &f = freed[bytes];
  if (f.empty()) {
    *p = aligned_alloc(256, (bytes + 255) / 256 * 256);
  } else {
    *p = f.back();
    f.pop_back();
  }
  blocks[*p] = bytes;
  return OK;
}
int hipFree(void *p) {
  if (any_capture()) return in_capture();
  auto b = blocks.find(p);
  if (b == blocks.end()) return p ? fail(1) : OK;
  freed[b->second].push_back(p);
  blocks.erase(b);
  return OK;
}
int hipHostMalloc(void **p, size_t bytes, unsigned) {
  *p = calloc(1, bytes);
  return OK;
}
int hipHostFree(void *p) {
  free(p);
  return OK;
}
int hipMemcpyAsync(void *dst, const void *src, size_t bytes, int, stream_t s) {
  ++copies;
  if (capturing[s]) recorded.push_back({dst, src, bytes});
  else memmove(dst, src, bytes);
  return OK;
}
int hipMemcpy2DAsync(void *, size_t, const void *, size_t, size_t, size_t, int, stream_t) { return OK; }
int hipStreamSynchronize(stream_t s) { return capturing[s] ? in_capture() : OK; }
int hipDeviceSynchronize() { return OK; }
int hipStreamIsCapturing(stream_t s, int *status) {
  *status = capturing[s];
  return OK;
}
int hipStreamCreateWithFlags(stream_t *s, unsigned) {
  *s = malloc(1);
  return OK;
}
int hipStreamDestroy(stream_t) { return OK; }
int hipStreamWaitEvent(stream_t, void *, unsigned) { return OK; }
int hipStreamBeginCapture(stream_t s, int) {
  capturing[s] = true;
  return OK;
}
int hipStreamEndCapture(stream_t s, void **g) {
  capturing[s] = false;
  *g = malloc(1);
  return OK;
}
int hipGraphInstantiate(void **e, void *, void *, char *, size_t) {
  *e = malloc(1);
  return OK;
}
int hipGraphLaunch(void *, stream_t) { return OK; }
int hipGraphDestroy(void *) { return OK; }
int hipGraphExecDestroy(void *) { return OK; }
int hipEventCreate(void **e) {
  *e = malloc(1);
  return OK;
}
int hipEventCreateWithFlags(void **e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void *) { return OK; }
int hipEventRecord(void *, stream_t) { return OK; }
int hipEventSynchronize(void *) { return OK; }
int hipEventElapsedTime(float *ms, void *, void *) {
  *ms = !launches.empty() && launches.back().name.find("part_sum") != std::string::npos ? cut_ms : 1.0f;
  return OK;
}
int hipGetDeviceCount(int *n) {
  *n = 1;
  return OK;
}
int hipSetDevice(int) { return OK; }
int hipGetDevicePropertiesR0600(void *, int) { return 1; }      // the library then takes its own architecture name
int hipGetSymbolAddress(void **p, const void *) {
  static void *scratch = aligned_alloc(256, size_t(8) << 20);
  *p = scratch;
  return OK;
}
const char *hipGetErrorString(int) { return "error"; }
int hipGetLastError() {
  const int e = last;
  last = OK;
  return e;
}

}  // extern "C"
