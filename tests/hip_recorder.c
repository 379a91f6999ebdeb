/* A stand-in for the HIP runtime (LD_PRELOAD): no GPU, launches are written down and cost the time that the test states. */
#include <stdint.h>
#include <stdio.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;

static struct { const void* host; const char* name; } kernels[4096];
static int n_kernels;
static struct { char name[96]; float ms, ms_repeated; } costs[64];
static int n_costs;
static char launches[1 << 20];
static size_t at;
static const void* last;
static float now;

/* For the tests: kernels whose name holds `name` cost `ms`, right after themselves `ms_repeated` (the first rule that fits). */
void recorder_cost(const char* name, float ms, float ms_repeated) {
  snprintf(costs[n_costs].name, sizeof costs[0].name, "%s", name);
  costs[n_costs].ms = ms;
  costs[n_costs++].ms_repeated = ms_repeated;
}
/* The mangled names launched since the last call, one a line. */
const char* recorder_launches(void) {
  launches[at] = 0;
  at = 0;
  return launches;
}

void** __hipRegisterFatBinary(const void* data) { static void* handle; (void)data; return &handle; }
void __hipUnregisterFatBinary(void** modules) { (void)modules; }
void __hipRegisterFunction(void** modules, const void* host, char* device, const char* name, unsigned limit, void* tid, void* bid,
                           dim3_t* block, dim3_t* grid, int* size) {
  (void)modules; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)size;
  if (n_kernels < 4096) { kernels[n_kernels].host = host; kernels[n_kernels++].name = name; }
}
void __hipRegisterVar(void** modules, void* var, char* host, char* device, int ext, size_t size, int constant, int global) {
  (void)modules; (void)var; (void)host; (void)device; (void)ext; (void)size; (void)constant; (void)global;
}
static struct { dim3_t grid, block; size_t lds; void* stream; } pushed;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) {
  pushed.grid = grid; pushed.block = block; pushed.lds = lds; pushed.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) {
  *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
  return 0;
}
int hipLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream) {
  (void)grid; (void)block; (void)args; (void)lds; (void)stream;
  const char* name = "?";
  for (int i = 0; i < n_kernels; ++i) if (kernels[i].host == f) name = kernels[i].name;
  for (int i = 0; i < n_costs; ++i)
    if (strstr(name, costs[i].name)) { now += f == last ? costs[i].ms_repeated : costs[i].ms; break; }
  last = f;
  if (at + strlen(name) + 2 < sizeof launches) at += (size_t)sprintf(launches + at, "%s\n", name);
  return 0;
}
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void* f, int attribute, int value) { (void)f; (void)attribute; (void)value; return 0; }
int hipGetDevice(int* device) { *device = 0; return 0; }
int hipGetSymbolAddress(void** p, const void* symbol) { (void)symbol; *p = (void*)0x1000; return 0; }
int hipEventCreate(void** e) { static float times[1024]; static int n; *e = &times[n++ % 1024]; return 0; }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipEventRecord(void* e, void* stream) { (void)stream; *(float*)e = now; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { *ms = *(float*)b - *(float*)a; return 0; }
