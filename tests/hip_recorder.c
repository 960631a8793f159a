/* A stand-in for the HIP runtime under the library's host code, for tests without a GPU: device memory
 * is address space that nothing reads, a launch is a line in a log.  Loaded with RTLD_GLOBAL before
 * the library, its symbols are found before those of the real runtime. */
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2 };

/* ---- what a test sets and reads ---- */
static size_t budget = SIZE_MAX, live;
static int capturing, device, pending;
static char log_text[1 << 16];
static size_t log_len;

void rec_budget(size_t bytes) { budget = bytes; }
void rec_capturing(int on) { capturing = on; }
void rec_device(int id) { device = id; }
void rec_pending(int error) { pending = error; }  /* what an earlier call of the program left behind */
size_t rec_live(void) { return live; }
const char* rec_log(void) { return log_text; }
void rec_clear(void) { log_len = 0; log_text[0] = 0; }

static void note(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  int w = vsnprintf(log_text + log_len, sizeof(log_text) - log_len, fmt, ap);
  va_end(ap);
  if (w > 0 && log_len + (size_t)w < sizeof(log_text)) log_len += (size_t)w;
}

/* ---- memory ---- */
static struct { char* p; size_t n; } blocks[4096];
static int n_blocks;
static char* next_address = (char*)(uintptr_t)(1ull << 40);

int hipMalloc(void** p, size_t n) {
  int slot = 0;
  while (slot < n_blocks && blocks[slot].n) ++slot;
  if (n > budget - (live < budget ? live : budget) || slot == 4096) {
    note("malloc-failed %zu\n", n);
    return pending = hipErrorOutOfMemory;
  }
  if (slot == n_blocks) ++n_blocks;
  *p = next_address;
  blocks[slot].p = next_address;
  blocks[slot].n = n;
  next_address += (n + 0xFFFFF) & ~(size_t)0xFFFFF;
  live += n;
  note("malloc %p %zu\n", *p, n);
  return hipSuccess;
}

int hipFree(void* p) {
  for (int i = 0; i < n_blocks; ++i)
    if (blocks[i].p == (char*)p && blocks[i].n) {
      live -= blocks[i].n;
      blocks[i].n = 0;
      note("free %p\n", p);
      return hipSuccess;
    }
  note("bad-free %p\n", p);
  return hipErrorInvalidValue;
}

/* ---- kernels ---- */
static struct { const void* f; char name[512]; } kernels[4096];
static int n_kernels;

void** __hipRegisterFatBinary(const void* data) { (void)data; return (void**)&n_kernels; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* a, char* b, int c, size_t d, int e, int f) {
  (void)m; (void)v; (void)a; (void)b; (void)c; (void)d; (void)e; (void)f;
}
void __hipRegisterFunction(void** m, const void* f, char* a, const char* name, unsigned b, void* c, void* d, void* e,
                           void* g, int* h) {
  (void)m; (void)a; (void)b; (void)c; (void)d; (void)e; (void)g; (void)h;
  if (n_kernels == 4096) return;
  kernels[n_kernels].f = f;
  snprintf(kernels[n_kernels++].name, sizeof(kernels[0].name), "%s", name);
}
static const char* name_of(const void* f) {
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].f == f) return kernels[i].name;
  return "?";
}

static struct { dim3 grid, block; size_t shared; void* stream; } config;
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void* stream) {
  config.grid = grid; config.block = block; config.shared = shared; config.stream = stream;
  return hipSuccess;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, void** stream) {
  *grid = config.grid; *block = config.block; *shared = config.shared; *stream = config.stream;
  return hipSuccess;
}
int hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t shared, void* stream) {
  (void)args; (void)stream;
  note("launch %s %u %u %u %u %zu %d\n", name_of(f), grid.x, grid.y, grid.z, block.x, shared, device);
  return hipSuccess;
}
int hipFuncSetAttribute(const void* f, int attr, int value) {
  (void)attr;
  note("lds-limit %s %d %d\n", name_of(f), value, device);
  return hipSuccess;
}

/* ---- the rest ---- */
int hipGetLastError(void) { const int e = pending; pending = hipSuccess; return e; }
int hipGetDeviceCount(int* n) { *n = 128; return hipSuccess; }
int hipGetDevice(int* id) { *id = device; return hipSuccess; }
int hipGetSymbolAddress(void** p, const void* symbol) { (void)symbol; *p = (void*)(uintptr_t)(1ull << 36); return hipSuccess; }
int hipStreamIsCapturing(void* stream, int* status) { (void)stream; *status = capturing ? 1 : 0; return hipSuccess; }
int hipStreamSynchronize(void* stream) { (void)stream; return hipSuccess; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* stream) {
  (void)d; (void)s; (void)n; (void)kind; (void)stream;
  return hipSuccess;
}
static uintptr_t next_event = 1;
int hipEventCreate(void** e) { *e = (void*)next_event++; return hipSuccess; }
int hipEventDestroy(void* e) { (void)e; return hipSuccess; }
int hipEventRecord(void* e, void* stream) { (void)stream; note("event %p\n", e); return hipSuccess; }
int hipEventSynchronize(void* e) { (void)e; return hipSuccess; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0.f; return hipSuccess; }
