// The HIP runtime calls that the library makes, without a GPU: "device" memory is host memory, a launch writes down its kernel's name, grid,
// workgroup and LDS bytes.  For tests of which kernels a call launches (test_dispatch.py); nothing is computed.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct {
  uint32_t x, y, z;
} Dim;
enum { MOST = 8192 };
static struct {
  const void *host;
  char *name;
} kernels[MOST];
static int nkernels, allocations;
static char text[1 << 16];
static size_t used;
static struct {
  Dim grid, block;
  size_t lds;
  void *stream;
} pushed;

int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void *stream) {
  pushed.grid = grid;
  pushed.block = block;
  pushed.lds = lds;
  pushed.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(Dim *grid, Dim *block, size_t *lds, void **stream) {
  *grid = pushed.grid;
  *block = pushed.block;
  *lds = pushed.lds;
  *stream = pushed.stream;
  return 0;
}
void **__hipRegisterFatBinary(const void *data) {
  static void *handle;
  return &handle;
}
void __hipRegisterFunction(void **modules, const void *host, char *device, const char *name, unsigned limit, void *tid, void *bid, void *block,
                           void *grid, int *wave) {
  if (nkernels < MOST) {
    kernels[nkernels].host = host;
    kernels[nkernels++].name = strdup(name);
  }
}
void __hipRegisterVar(void **modules, void *var, char *host, char *device, int ext, size_t size, int constant, int global) {}
void __hipUnregisterFatBinary(void **modules) {}
int hipMalloc(void **p, size_t n) {
  *p = malloc(n ? n : 1);
  ++allocations;
  return *p ? 0 : 2;
}
int hipFree(void *p) {
  free(p);
  return 0;
}
int hipMemcpy(void *to, const void *from, size_t n, int kind) {
  memcpy(to, from, n);
  return 0;
}
int hipMemcpyAsync(void *to, const void *from, size_t n, int kind, void *stream) { return hipMemcpy(to, from, n, kind); }
int hipStreamSynchronize(void *stream) { return 0; }
int hipFuncSetAttribute(const void *f, int attribute, int value) { return 0; }
int hipGetDevice(int *d) {
  *d = 0;
  return 0;
}
int hipGetSymbolAddress(void **p, const void *symbol) { return 1; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { return "no GPU"; }
int hipLaunchKernel(const void *f, Dim grid, Dim block, void **args, size_t lds, void *stream) {
  const char *name = "?";
  for (int k = 0; k < nkernels; ++k)
    if (kernels[k].host == f) name = kernels[k].name;
  if (used + strlen(name) + 64 < sizeof text)
    used += (size_t)sprintf(text + used, "%s %u %u %u %zu\n", name, grid.x, grid.y, block.x, lds);
  return 0;
}

// what was launched since the last call; *n: allocations since then
const char *stub_take(int *n) {
  *n = allocations;
  allocations = 0;
  text[used] = 0;
  used = 0;
  return text;
}
