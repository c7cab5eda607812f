/* A HIP runtime without a GPU, for tests of the host code that plans launches: memory is
 * host memory, kernels do not run, and each launch is logged with its device name, grid
 * and stream.  Loaded with RTLD_GLOBAL before libmhd.so, whose calls then bind to it.
 * The time between two events is what fake_time_of() says of the last kernel logged. */
#include <stddef.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3;
enum { MAXK = 4096, MAXLOG = 1 << 16 };

static struct { const void* host; const char* name; } kernels[MAXK];
static int nkernels;
static struct { const char* name; unsigned grid; } launched[MAXLOG];
static int nlaunched;
static float (*time_of)(const char* name, unsigned grid);
static struct { dim3 grid, block; size_t lds; void* stream; } pending;

void fake_time_of(float (*f)(const char*, unsigned)) { time_of = f; }
void fake_clear(void) { nlaunched = 0; }
int fake_count(void) { return nlaunched; }
const char* fake_name(int i) { return launched[i].name; }
unsigned fake_grid(int i) { return launched[i].grid; }

void** __hipRegisterFatBinary(const void* data) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void** h) {}
void __hipRegisterFunction(void** h, const void* host, char* dev, const char* name, unsigned limit,
                           void* tid, void* bid, void* bdim, void* gdim, int* wsize) {
  if (nkernels < MAXK) { kernels[nkernels].host = host; kernels[nkernels++].name = name; }
}
void __hipRegisterVar(void** h, void* var, char* a, char* b, int ext, size_t size, int c, int g) {}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream) {
  pending.grid = grid; pending.block = block; pending.lds = lds; pending.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) {
  *grid = pending.grid; *block = pending.block; *lds = pending.lds; *stream = pending.stream;
  return 0;
}
int hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, void* stream) {
  for (int i = 0; i < nkernels; ++i)
    if (kernels[i].host == f && nlaunched < MAXLOG) {
      launched[nlaunched].name = kernels[i].name;
      launched[nlaunched++].grid = grid.x;
    }
  return 0;
}
int hipFuncSetAttribute(const void* f, int attr, int value) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int d) { return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void** p, const void* symbol) { return 1; }
int hipHostMalloc(void** p, size_t size, unsigned flags) { *p = malloc(size); return *p ? 0 : 2; }
int hipMemGetAddressRange(void** base, size_t* size, void* p) { return 1; }
int hipPointerGetAttributes(void* attributes, const void* p) { return 1; }
int hipMemcpy(void* dst, const void* src, size_t n, int kind) { memcpy(dst, src, n); return 0; }
int hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void* stream) {
  memcpy(dst, src, n);
  return 0;
}
int hipStreamSynchronize(void* stream) { return 0; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* stream) { return 0; }
int hipEventSynchronize(void* e) { return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) {
  *ms = nlaunched && time_of ? time_of(launched[nlaunched - 1].name, launched[nlaunched - 1].grid) : 1.0f;
  return 0;
}
