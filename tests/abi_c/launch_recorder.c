/* What the library launches for given arguments, without a GPU: the HIP runtime functions that it calls are defined here (an
 * executable's symbols come before those of the shared libraries), and print each launch instead of starting it.  One call per line on
 * stdin: the entry point's name and the fields of sage_attn_args that differ from zero, as name=value; q, k, v, out and the workspace
 * are set unless the line sets them.  Answers one line per launch, "launch <kernel, mangled> <grid x> <y> <z> <block x>", then
 * "status <result>".  Built and run by tests/launch_recorder.py. */
#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "sage_attn.h"

enum { MAX_KERNELS = 4096 };
static struct { const void* stub; const char* name; } kernels[MAX_KERNELS];
static int n_kernels;
static dim3 call_grid, call_block;

static void* modules[4];
void** __hipRegisterFatBinary(const void* data) { (void)data; return modules; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* var, char* host, const char* dev, int ext, size_t size, int constant, int global) {
  (void)m; (void)var; (void)host; (void)dev; (void)ext; (void)size; (void)constant; (void)global;
}
void __hipRegisterFunction(void** m, const void* stub, char* dev, const char* name, unsigned limit, void* tid, void* bid, void* bdim,
                           void* gdim, int* wsize) {
  (void)m; (void)dev; (void)limit; (void)tid; (void)bid; (void)bdim; (void)gdim; (void)wsize;
  if (n_kernels == MAX_KERNELS) abort();
  kernels[n_kernels].stub = stub;
  kernels[n_kernels++].name = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
  (void)shared; (void)s;
  call_grid = grid; call_block = block;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* s) {
  *grid = call_grid; *block = call_block; *shared = 0; *s = 0;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* stub, dim3 grid, dim3 block, void** args, size_t shared, hipStream_t s) {
  (void)args; (void)shared; (void)s;
  const char* name = "unknown";
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].stub == stub) name = kernels[i].name;
  printf("launch %s %u %u %u %u\n", name, grid.x, grid.y, grid.z, block.x);
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int d) { (void)d; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { (void)n; *p = (void*)(uintptr_t)4096; return hipSuccess; }
hipError_t hipFree(void* p) { (void)p; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* sym) { (void)sym; *p = (void*)(uintptr_t)4096; return hipSuccess; }

#define INT_FIELD(f) { #f, offsetof(sage_attn_args, f), 0 }
#define PTR_FIELD(f) { #f, offsetof(sage_attn_args, f), 1 }
static const struct { const char* name; size_t off; int pointer; } fields[] = {
    INT_FIELD(B), INT_FIELD(H), INT_FIELD(H_kv), INT_FIELD(N), INT_FIELD(d), INT_FIELD(causal), INT_FIELD(mode), INT_FIELD(dtype),
    INT_FIELD(flags), INT_FIELD(group_map), INT_FIELD(N_kv), INT_FIELD(layout), INT_FIELD(pv_format), INT_FIELD(kv_splits),
    PTR_FIELD(q), PTR_FIELD(k), PTR_FIELD(v), PTR_FIELD(out), PTR_FIELD(workspace), PTR_FIELD(cu_seqlens_q),
    PTR_FIELD(cu_seqlens_k), PTR_FIELD(lse), PTR_FIELD(k_mean_in), PTR_FIELD(v_scale_in), PTR_FIELD(workspace_bytes)};   /* (a size_t) */

static int set_field(sage_attn_args* a, const char* name, long long value) {
  for (size_t i = 0; i < sizeof fields / sizeof fields[0]; ++i) {
    if (strcmp(fields[i].name, name) != 0) continue;
    char* p = (char*)a + fields[i].off;
    if (fields[i].pointer) *(void**)p = (void*)(uintptr_t)value;
    else *(int*)p = (int)value;
    return 1;
  }
  return 0;
}

int main(void) {
  char line[1024];
  while (fgets(line, sizeof line, stdin)) {
    char* word = strtok(line, " \n");
    if (!word) continue;
    sage_attn_args a;
    memset(&a, 0, sizeof a);
    a.q = a.k = a.v = a.out = a.workspace = (void*)(uintptr_t)4096;
    a.workspace_bytes = (size_t)-1;
    const char* entry = word;
    while ((word = strtok(NULL, " \n")) != NULL) {
      char* eq = strchr(word, '=');
      if (!eq) { fprintf(stderr, "no value in %s\n", word); return 2; }
      *eq = 0;
      if (!set_field(&a, word, atoll(eq + 1))) { fprintf(stderr, "no field %s\n", word); return 2; }
    }
    int st;
    if (strcmp(entry, "sage_attn_fwd_ex") == 0) st = sage_attn_fwd_ex(&a);
    else if (strcmp(entry, "sage_attn_fwd_static") == 0) st = sage_attn_fwd_static(&a);
    else if (strcmp(entry, "sage_attn_prologue") == 0) st = sage_attn_prologue(&a);
    else if (strcmp(entry, "sage_attn_kv_stats") == 0) st = sage_attn_kv_stats(&a, (void*)(uintptr_t)4096, (void*)(uintptr_t)4096);
    else { fprintf(stderr, "no entry point %s\n", entry); return 2; }
    printf("status %d\n", st);
  }
  return 0;
}
