/* Stand-in for the HIP runtime symbols that libpquant uses, for tests without a GPU: a launch records the kernel's name and
   grid and returns success, so that a whole library call runs its host side and nothing else.  Loaded with RTLD_GLOBAL ahead
   of the library (launch_trace.py). */
#include <stddef.h>
#include <stdint.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct { const char* name; dim3_t grid; } launch_t;

enum { MAX_KERNELS = 4096, MAX_LAUNCHES = 4096 };
static struct { const void* fn; const char* name; } kernels[MAX_KERNELS];
static int n_kernels, n_launches;
static launch_t launches[MAX_LAUNCHES];
static dim3_t cfg_grid, cfg_block;
static size_t cfg_lds;
static void* cfg_stream;
static char memory[64];

void trace_reset(void) { n_launches = 0; }
int trace_count(void) { return n_launches; }
const char* trace_name(int i) { return launches[i].name; }
uint32_t trace_grid(int i, int axis) { return axis == 0 ? launches[i].grid.x : axis == 1 ? launches[i].grid.y : launches[i].grid.z; }

void** __hipRegisterFatBinary(const void* data) { static void* module; (void)data; return &module; }
void __hipUnregisterFatBinary(void** module) { (void)module; }
void __hipRegisterVar(void** module, void* var, char* host, char* dev, int ext, size_t size, int constant, int global) {
  (void)module; (void)var; (void)host; (void)dev; (void)ext; (void)size; (void)constant; (void)global;
}
void __hipRegisterFunction(void** module, const void* fn, char* dev_fn, const char* name, unsigned limit, void* a, void* b, void* c, void* d,
                           int* e) {
  (void)module; (void)dev_fn; (void)limit; (void)a; (void)b; (void)c; (void)d; (void)e;
  if (n_kernels < MAX_KERNELS) { kernels[n_kernels].fn = fn; kernels[n_kernels++].name = name; }
}
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) {
  cfg_grid = grid; cfg_block = block; cfg_lds = lds; cfg_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) {
  *grid = cfg_grid; *block = cfg_block; *lds = cfg_lds; *stream = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void* fn, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream) {
  (void)block; (void)args; (void)lds; (void)stream;
  if (n_launches >= MAX_LAUNCHES) return 1;
  launches[n_launches].name = "?";
  launches[n_launches].grid = grid;
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].fn == fn) launches[n_launches].name = kernels[i].name;
  ++n_launches;
  return 0;
}
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { (void)e; return "stand-in"; }
int hipFuncSetAttribute(const void* fn, int attr, int value) { (void)fn; (void)attr; (void)value; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetSymbolAddress(void** p, const void* symbol) { (void)symbol; *p = memory; return 0; }
