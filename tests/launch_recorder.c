/* A HIP runtime that launches nothing: it hands every kernel launch to a callback.  Loaded ahead of the library (in a
 * process of its own), it shows on a machine without a GPU which kernels a call would run. */
#include <stddef.h>
#include <stdint.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef void (*launch_fn)(const void *stub, const uint32_t *grid, const uint32_t *block, size_t lds, void **args);
typedef void (*kernel_fn)(const void *stub, const char *name);

enum { MAX_KERNELS = 1024 };
static const void *stubs[MAX_KERNELS];
static const char *names[MAX_KERNELS];
static int n_kernels;
static launch_fn on_launch;
static dim3 next_grid, next_block;
static size_t next_lds;
static void *next_stream, *module;

void recorder_kernels(kernel_fn each) { for (int i = 0; i < n_kernels; ++i) each(stubs[i], names[i]); }
void recorder_on_launch(launch_fn fn) { on_launch = fn; }

void **__hipRegisterFatBinary(const void *data) { (void)data; return &module; }
void __hipUnregisterFatBinary(void **modules) { (void)modules; }
void __hipRegisterVar(void **modules, void *var, char *host, char *name, int ext, size_t size, int constant, int global) {
  (void)modules; (void)var; (void)host; (void)name; (void)ext; (void)size; (void)constant; (void)global;
}
void __hipRegisterFunction(void **modules, const void *stub, char *host, const char *name, unsigned limit, void *tid,
                           void *bid, dim3 *block, dim3 *grid, int *warp) {
  (void)modules; (void)host; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)warp;
  if (n_kernels < MAX_KERNELS) { stubs[n_kernels] = stub; names[n_kernels++] = name; }
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream) {
  next_grid = grid; next_block = block; next_lds = lds; next_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream) {
  *grid = next_grid; *block = next_block; *lds = next_lds; *stream = next_stream;
  return 0;
}
int hipLaunchKernel(const void *stub, dim3 grid, dim3 block, void **args, size_t lds, void *stream) {
  (void)stream;
  const uint32_t g[3] = {grid.x, grid.y, grid.z}, b[3] = {block.x, block.y, block.z};
  if (on_launch) on_launch(stub, g, b, lds, args);
  return 0;
}
int hipFuncSetAttribute(const void *stub, int attr, int value) { (void)stub; (void)attr; (void)value; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetDevice(int *device) { *device = 0; return 0; }
