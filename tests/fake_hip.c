/* A HIP runtime of two devices without kernels, for tests of the library's host part on the CPU.
 * "Device" memory is host memory, launches do nothing but are counted by the device they go to, copies are
 * made at once.  As in HIP, a stream and an event belong to the device that was current when they were made
 * (the null stream to the current one), an event is recorded on a stream of its own device only, and a launch has fewer
 * than 2^32 threads along each axis. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
struct on { int device; };
enum { kDevices = 2, kInvalidValue = 1, kInvalidConfiguration = 9, kInvalidDevice = 101, kInvalidHandle = 400 };

static __thread int current;
static __thread struct { dim3 grid, block; size_t shared; void* stream; } config;
static int launched[kDevices];
static struct { const void* f; char name[120]; int launched; uint64_t blocks; } kernels[256];
static int n_kernels;
static uint32_t row_total;          /* what row_total_kernel finds */
static uint32_t units;              /* of every diagonal, as scan_units_kernel finds them */
static __thread int last_error;

static int device_of(void* stream) { return stream ? ((struct on*)stream)->device : current; }
static int make(void** out) {
  struct on* s = malloc(sizeof *s);
  s->device = current;
  *out = s;
  return 0;
}

int fake_launches(int device) { return __atomic_load_n(&launched[device], __ATOMIC_SEQ_CST); }
/* launches of the kernels whose (mangled) name holds `part`, since the last call with this part */
int fake_launches_of(const char* part) {
  int n = 0;
  for (int i = 0; i < n_kernels; i++) if (strstr(kernels[i].name, part)) n += __atomic_exchange_n(&kernels[i].launched, 0, __ATOMIC_SEQ_CST);
  return n;
}
/* and their workgroups */
uint64_t fake_blocks_of(const char* part) {
  uint64_t n = 0;
  for (int i = 0; i < n_kernels; i++) if (strstr(kernels[i].name, part)) n += __atomic_exchange_n(&kernels[i].blocks, 0, __ATOMIC_SEQ_CST);
  return n;
}
void fake_row_total(uint32_t n) { row_total = n; }
void fake_units(uint32_t n) { units = n; }

int hipGetDevice(int* d) { *d = current; return 0; }
int hipSetDevice(int d) { if (d < 0 || d >= kDevices) return kInvalidDevice; current = d; return 0; }
int hipGetLastError(void) { int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int e) { return e == kInvalidHandle ? "invalid resource handle" : "error"; }

int hipStreamCreateWithFlags(void** s, unsigned flags) { (void)flags; return make(s); }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned flags) { (void)s; (void)flags; return e ? 0 : kInvalidHandle; }
int hipEventCreate(void** e) { return make(e); }
int hipEventCreateWithFlags(void** e, unsigned flags) { (void)flags; return make(e); }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* s) { return ((struct on*)e)->device == device_of(s) ? 0 : kInvalidHandle; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0; return 0; }

static int zeroed(void** p, size_t n) {
  if (posix_memalign(p, 256, n ? n : 1)) return 2;
  memset(*p, 0, n);
  return 0;
}
int hipMalloc(void** p, size_t n) { return zeroed(p, n); }
int hipFree(void* p) { free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned flags) { (void)flags; return zeroed(p, n); }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemcpy(void* to, const void* from, size_t n, int kind) { (void)kind; memcpy(to, from, n); return 0; }
int hipMemcpyAsync(void* to, const void* from, size_t n, int kind, void* s) { (void)s; return hipMemcpy(to, from, n, kind); }
int hipMemsetAsync(void* p, int v, size_t n, void* s) { (void)s; memset(p, v, n); return 0; }
int hipGetSymbolAddress(void** p, const void* symbol) { (void)symbol; *p = 0; return kInvalidValue; }

int hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t shared, void* s) {
  (void)shared;
  if ((uint64_t)grid.x * block.x >> 32 || (uint64_t)grid.y * block.y >> 32 || (uint64_t)grid.z * block.z >> 32) return last_error = kInvalidConfiguration;
  __atomic_add_fetch(&launched[device_of(s)], 1, __ATOMIC_SEQ_CST);
  for (int i = 0; i < n_kernels; i++) {
    if (kernels[i].f != f) continue;
    __atomic_add_fetch(&kernels[i].launched, 1, __ATOMIC_SEQ_CST);
    __atomic_add_fetch(&kernels[i].blocks, (uint64_t)grid.x * grid.y * grid.z, __ATOMIC_SEQ_CST);
    if (strstr(kernels[i].name, "row_total_kernel")) **(uint32_t**)args[2] = row_total;
    if (strstr(kernels[i].name, "scan_units_kernel")) {
      const uint32_t diagonals = *(uint32_t*)args[1] + *(uint32_t*)args[2] - 1;
      for (uint32_t d = 0; d <= diagonals; d++) (*(uint32_t**)args[6])[d] = d * units;
    }
  }
  return 0;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void* s) {
  config.grid = grid; config.block = block; config.shared = shared; config.stream = s;
  return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, void** s) {
  *grid = config.grid; *block = config.block; *shared = config.shared; *s = config.stream;
  return 0;
}
void** __hipRegisterFatBinary(const void* data) { static void* handle; (void)data; return &handle; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterFunction(void** h, const void* f, char* device_name, const char* name, unsigned threads, void* tid, void* bid, void* block,
                           void* grid, int* warp) {
  (void)h; (void)device_name; (void)threads; (void)tid; (void)bid; (void)block; (void)grid; (void)warp;
  if (n_kernels == 256) abort();
  kernels[n_kernels].f = f;
  strncpy(kernels[n_kernels++].name, name, sizeof kernels[0].name - 1);
}
void __hipRegisterVar(void** h, void* var, char* host_name, char* device_name, int ext, size_t size, int constant, int global) {
  (void)h; (void)var; (void)host_name; (void)device_name; (void)ext; (void)size; (void)constant; (void)global;
}
