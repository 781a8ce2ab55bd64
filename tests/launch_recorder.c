/* The HIP runtime calls of the library without a GPU: launches are written down, nothing runs.  Loaded ahead of the library
 * (RTLD_GLOBAL), so that its symbols are found before the runtime's. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef struct { char kernel[192]; uint32_t grid[3], block; uint32_t lds; } launch_t;

#define MAX_KERNELS 4096
#define MAX_LAUNCHES 256
static const void* stub_of[MAX_KERNELS];
static const char* name_of[MAX_KERNELS];
static int kernels, launches;
static launch_t list[MAX_LAUNCHES];
static dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static void* cfg_stream;

int recorded(void) { return launches; }
const launch_t* launch_at(int i) { return &list[i]; }
void forget(void) { launches = 0; }

void** __hipRegisterFatBinary(const void* data) { static void* handle; (void)data; return &handle; }
void __hipUnregisterFatBinary(void** modules) { (void)modules; }
void __hipRegisterFunction(void** modules, const void* stub, char* device, const char* name, unsigned threads, void* tid, void* bid,
                           dim3* block, dim3* grid, int* wsize) {
    (void)modules; (void)device; (void)threads; (void)tid; (void)bid; (void)block; (void)grid; (void)wsize;
    if (kernels < MAX_KERNELS) { stub_of[kernels] = stub; name_of[kernels++] = name; }
}
void __hipRegisterVar(void** modules, void* var, char* host, char* name, int ext, size_t size, int constant, int global) {
    (void)modules; (void)var; (void)host; (void)name; (void)ext; (void)size; (void)constant; (void)global;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream) {
    cfg_grid = grid; cfg_block = block; cfg_lds = lds; cfg_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) {
    *grid = cfg_grid; *block = cfg_block; *lds = cfg_lds; *stream = cfg_stream;
    return 0;
}
int hipLaunchKernel(const void* stub, dim3 grid, dim3 block, void** args, size_t lds, void* stream) {
    (void)args; (void)stream;
    if (launches == MAX_LAUNCHES) return 1;
    launch_t* l = &list[launches++];
    l->kernel[0] = 0;
    for (int i = 0; i < kernels; ++i)
        if (stub_of[i] == stub) snprintf(l->kernel, sizeof l->kernel, "%s", name_of[i]);
    l->grid[0] = grid.x; l->grid[1] = grid.y; l->grid[2] = grid.z;
    l->block = block.x * block.y * block.z;
    l->lds = (uint32_t)lds;
    return 0;
}
int hipFuncSetAttribute(const void* stub, int attr, int value) { (void)stub; (void)attr; (void)value; return 0; }
int hipGetDevice(int* device) { *device = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void** address, const void* symbol) { *address = (void*)symbol; return 0; }
