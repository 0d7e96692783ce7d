/* The entry points of the HIP runtime that the library uses, for a process without a device: one device of 256 compute units and 160 KiB
 * of LDS each, on which every launch succeeds without running.  Writes a line per kernel launch and per kernel attribute to the file
 * named by RECORD.  Loaded into the global scope before the library, it answers in the runtime's place. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
static struct { const void *handle; char name[512]; } kernels[512];
static int n_kernels;
static char scratch[64];

static const char *name_of(const void *handle) {
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].handle == handle) return kernels[i].name;
  return "?";
}
static FILE *record(void) {
  static FILE *f;
  if (f == NULL) f = fopen(getenv("RECORD"), "w");
  return f;
}

void **__hipRegisterFatBinary(const void *data) { (void)data; static void *module; return &module; }
void __hipUnregisterFatBinary(void **module) { (void)module; }
void __hipRegisterFunction(void **module, const void *handle, char *device, const char *name, unsigned limit, void *tid, void *bid, void *block,
                           void *grid, int *size) {
  (void)module; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)size;
  kernels[n_kernels].handle = handle;
  strncpy(kernels[n_kernels++].name, name, 511);
}
void __hipRegisterVar(void **module, void *var, char *host, char *device, int ext, size_t size, int constant, int global) {
  (void)module; (void)var; (void)host; (void)device; (void)ext; (void)size; (void)constant; (void)global;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream) { (void)grid; (void)block; (void)lds; (void)stream; return 1; }
int hipGetDevice(int *device) { *device = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipDeviceGetAttribute(int *value, int attribute, int device) { (void)attribute; (void)device; *value = 256; return 0; }
int hipGetSymbolAddress(void **address, const void *symbol) { (void)symbol; *address = scratch - (uintptr_t)scratch % 16 + 16; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *blocks, const void *handle, int threads, size_t lds) {
  (void)handle;
  const int by_lds = lds > 0 ? (int)(163840 / lds) : 8, by_threads = 512 / threads;
  *blocks = by_lds < by_threads ? by_lds : by_threads;
  return 0;
}
int hipFuncSetAttribute(const void *handle, int attribute, int value) {
  fprintf(record(), "attribute %s %d %d\n", name_of(handle), attribute, value);
  return 0;
}
int hipLaunchKernel(const void *handle, dim3 grid, dim3 block, void **args, size_t lds, void *stream) {
  (void)args; (void)stream;
  fprintf(record(), "launch %s %u %u %zu\n", name_of(handle), grid.x, block.x, lds);
  fflush(record());
  return 0;
}
