/* Stand-in for the HIP runtime calls that libdpse makes, for host tests
 * without a GPU: allocations are address ranges that nothing reads or writes,
 * launches are recorded (kernel name, grid, work-group, dynamic LDS, the
 * leading bytes of the first argument) and run nothing.  Loaded with global
 * symbols before libdpse.so, whose calls then come here. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef int err_t;
typedef struct { uint32_t x, y, z; } dim3_t;

enum { MAX_FN = 1024, MAX_ALLOC = 4096, MAX_LAUNCH = 8192, ARG_WORDS = 192 };
static int ncu = 263; /* (a prime: sizes in lines per compute unit are told from the others) */

static struct { const void* host; const char* name; } fn[MAX_FN];
static int nfn;
static struct { uint64_t base, bytes; } alloc_[MAX_ALLOC];
static int nalloc;
static uint64_t next_addr = 1ull << 44;
typedef struct {
  const char* name;
  uint32_t grid[3], block[3];
  uint64_t lds;
  uint64_t arg[ARG_WORDS];
} launch_t;
static launch_t launch[MAX_LAUNCH];
static int nlaunch;

/* ---- reading the record */
int rec_ncu(void) { return ncu; }
void rec_set_ncu(int n) { ncu = n; }
int rec_launches(void) { return nlaunch; }
const launch_t* rec_launch(int k) { return &launch[k]; }
void rec_clear(void) { nlaunch = 0; }
/* bytes of the allocation that starts at p (0: none) */
uint64_t rec_bytes(uint64_t p) {
  for (int k = 0; k < nalloc; ++k)
    if (alloc_[k].base == p) return alloc_[k].bytes;
  return 0;
}

/* ---- memory */
err_t hipMalloc(void** p, size_t n) {
  if (nalloc == MAX_ALLOC) return 2;
  alloc_[nalloc].base = next_addr;
  alloc_[nalloc++].bytes = n;
  *p = (void*)next_addr;
  next_addr += (n + 511) & ~(uint64_t)255;
  return 0;
}
err_t hipFree(void* p) {
  for (int k = 0; k < nalloc; ++k)
    if (alloc_[k].base == (uint64_t)p) {
      alloc_[k] = alloc_[--nalloc];
      return 0;
    }
  return 1;
}
err_t hipHostMalloc(void** p, size_t n, unsigned f) {
  (void)f;
  *p = calloc(1, n);
  return *p ? 0 : 2;
}
err_t hipHostFree(void* p) {
  free(p);
  return 0;
}
err_t hipMemcpy(void* d, const void* s, size_t n, int k) { (void)d; (void)s; (void)n; (void)k; return 0; }
err_t hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { (void)d; (void)s; (void)n; (void)k; (void)st; return 0; }
err_t hipMemset(void* d, int v, size_t n) { (void)d; (void)v; (void)n; return 0; }
err_t hipGetSymbolAddress(void** p, const void* s) { (void)s; return hipMalloc(p, 1 << 23); }

/* ---- device, events, streams */
err_t hipGetDevice(int* d) { *d = 0; return 0; }
err_t hipSetDevice(int d) { (void)d; return 0; }
err_t hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = ncu; return 0; }
err_t hipDeviceSynchronize(void) { return 0; }
err_t hipStreamSynchronize(void* s) { (void)s; return 0; }
err_t hipGetLastError(void) { return 0; }
const char* hipGetErrorString(err_t e) { return e ? "error" : "success"; }
err_t hipEventCreate(void** e) { *e = (void*)1; return 0; }
err_t hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = (void*)1; return 0; }
err_t hipEventDestroy(void* e) { (void)e; return 0; }
err_t hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
err_t hipEventSynchronize(void* e) { (void)e; return 0; }
err_t hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0; return 0; }

/* ---- launches */
void** __hipRegisterFatBinary(const void* data) {
  static void* handle;
  (void)data;
  return &handle;
}
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned limit, void* tid, void* bid,
                           void* bdim, void* gdim, int* wsize) {
  (void)m; (void)dev; (void)limit; (void)tid; (void)bid; (void)bdim; (void)gdim; (void)wsize;
  if (nfn < MAX_FN) {
    fn[nfn].host = host;
    fn[nfn++].name = name;
  }
}
void __hipRegisterVar(void** m, void* var, char* host, char* name, int ext, size_t size, int con, int global) {
  (void)m; (void)var; (void)host; (void)name; (void)ext; (void)size; (void)con; (void)global;
}
static struct { dim3_t grid, block; size_t lds; void* stream; } conf;
err_t __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) {
  conf.grid = grid;
  conf.block = block;
  conf.lds = lds;
  conf.stream = stream;
  return 0;
}
err_t __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) {
  *grid = conf.grid;
  *block = conf.block;
  *lds = conf.lds;
  *stream = conf.stream;
  return 0;
}
err_t hipLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream) {
  (void)stream;
  if (nlaunch == MAX_LAUNCH) return 2;
  launch_t* l = &launch[nlaunch++];
  l->name = "?";
  for (int k = 0; k < nfn; ++k)
    if (fn[k].host == f) l->name = fn[k].name;
  l->grid[0] = grid.x; l->grid[1] = grid.y; l->grid[2] = grid.z;
  l->block[0] = block.x; l->block[1] = block.y; l->block[2] = block.z;
  l->lds = lds;
  /* (the arguments lie in the caller's stack frames, with more stack above
   * them than is copied) */
  if (args && args[0]) memcpy(l->arg, args[0], sizeof(l->arg));
  return 0;
}
