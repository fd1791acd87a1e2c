/* A stand-in for the HIP calls that the library makes, for host-side tests
 * without a GPU: device memory is host memory, kernels do nothing and are
 * counted, and a copy from pinned memory reads its source as late as it may (at
 * the next wait), so that a source rewritten before that is noticed. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;

enum { MAXP = 1024, MAXC = 256 };
static struct { char* at; size_t n; } pinned[MAXP];
static struct { char *dst, *seen; const char* src; size_t n; } pending[MAXC];
static int npinned, npending;
static long rewritten, launches, blocks;
static dim3_t cfg_grid, cfg_block;
static size_t cfg_lds;
static void* cfg_stream;

long fake_rewritten(void) { return rewritten; }
long fake_launches(void) { return launches; }
long fake_blocks(void) { return blocks; }

static void complete(void) {
  for (int i = 0; i < npending; ++i) {
    if (memcmp(pending[i].seen, pending[i].src, pending[i].n)) ++rewritten;
    memcpy(pending[i].dst, pending[i].src, pending[i].n);
    free(pending[i].seen);
  }
  npending = 0;
}

static int is_pinned(const void* p) {
  for (int i = 0; i < npinned; ++i)
    if ((const char*)p >= pinned[i].at && (const char*)p < pinned[i].at + pinned[i].n) return 1;
  return 0;
}

int hipMalloc(void** p, size_t n) { return posix_memalign(p, 256, n ? n : 256) ? 2 : 0; }
int hipFree(void* p) { free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned flags) {
  (void)flags;
  if (npinned == MAXP || posix_memalign(p, 256, n)) return 2;
  pinned[npinned].at = *p;
  pinned[npinned++].n = n;
  return 0;
}
int hipHostFree(void* p) {
  complete();
  for (int i = 0; i < npinned; ++i)
    if (pinned[i].at == p) pinned[i] = pinned[--npinned];
  free(p);
  return 0;
}
int hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void* stream) {
  (void)stream;
  if (kind == 1 && is_pinned(src)) {
    if (npending == MAXC) return 2;
    pending[npending].dst = dst;
    pending[npending].src = src;
    pending[npending].n = n;
    pending[npending].seen = malloc(n);
    memcpy(pending[npending++].seen, src, n);
  } else {
    memcpy(dst, src, n);
  }
  return 0;
}
int hipMemsetAsync(void* p, int v, size_t n, void* s) { (void)s; memset(p, v, n); return 0; }
int hipStreamSynchronize(void* s) { (void)s; complete(); return 0; }
int hipStreamIsCapturing(void* s, int* st) { (void)s; *st = 0; return 0; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void* e) { (void)e; complete(); return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 1.f; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetSymbolAddress(void** p, const void* sym) { static char scratch[256]; (void)sym; *p = scratch; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) {
  cfg_grid = grid;
  cfg_block = block;
  cfg_lds = lds;
  cfg_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) {
  *grid = cfg_grid;
  *block = cfg_block;
  *lds = cfg_lds;
  *stream = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream) {
  (void)f, (void)block, (void)args, (void)lds, (void)stream;
  ++launches;
  blocks += (long)grid.x * grid.y * grid.z;
  return 0;
}
