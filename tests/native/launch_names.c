/* Loaded in front of the HIP runtime: a kernel launch writes the kernel's name to stderr and launches nothing, so that a machine
 * without a GPU can say which kernels a call takes.  Test infrastructure, not product code. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
#include <stdio.h>

typedef struct { unsigned x, y, z; } Dim3;

static Dim3 grid_, block_;
static size_t lds_;

int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
    (void)stream;
    grid_ = grid, block_ = block, lds_ = lds;
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
    *grid = grid_, *block = block_, *lds = lds_, *stream = NULL;
    return 0;
}
int hipLaunchKernel(const void* kernel, Dim3 grid, Dim3 block, void** args, size_t lds, void* stream) {
    Dl_info info;
    const int known = dladdr(kernel, &info) != 0 && info.dli_saddr == kernel && info.dli_sname != NULL;
    (void)grid, (void)block, (void)args, (void)lds, (void)stream;
    fprintf(stderr, "launch %s\n", known ? info.dli_sname : "?");
    return 0;
}
int hipFuncSetAttribute(const void* kernel, int attribute, int value) { (void)kernel, (void)attribute, (void)value; return 0; }
int hipGetLastError(void) { return 0; }
int hipPeekAtLastError(void) { return 0; }
