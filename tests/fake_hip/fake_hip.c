/* A device of host memory for the CPU tests of the library's host code: the HIP calls it makes, with
 * allocations that can be made to fail.  Kernels do not run (hipLaunchKernel does nothing), so only what
 * happens before the first result of one is read can be tested. */
#include <stdlib.h>
#include <string.h>

enum { kOk = 0, kOutOfMemory = 2 };
static int calls, first_bad, last_bad; /* allocations [first_bad, last_bad] fail, counted from 1 */
static size_t refuse_from, refuse_to; /* and those of refuse_from to refuse_to bytes */
static long live;

void fake_hip_fail(int first, int last)
{
    calls = 0;
    first_bad = first;
    last_bad = last;
}
void fake_hip_refuse(size_t from, size_t to)
{
    refuse_from = from;
    refuse_to = to;
}
int fake_hip_allocations(void) { return calls; }
long fake_hip_live(void) { return live; }

static size_t free_bytes = 100, total_bytes = 100;
static int capturing;
void fake_hip_memory(size_t free_now, size_t total) { free_bytes = free_now; total_bytes = total; }
void fake_hip_capture(int on) { capturing = on; }

int hipMemGetInfo(size_t *f, size_t *t) { *f = free_bytes; *t = total_bytes; return kOk; }
int hipStreamIsCapturing(void *s, int *status) { (void)s; *status = capturing; return kOk; }
int hipThreadExchangeStreamCaptureMode(int *mode) { (void)mode; return kOk; }
int hipGetDeviceCount(int *n) { *n = 1; return kOk; }
int hipGetDevice(int *d) { *d = 0; return kOk; }
int hipSetDevice(int d) { (void)d; return kOk; }
int hipGetLastError(void) { return kOk; }
int hipDeviceSynchronize(void) { return kOk; }
int hipStreamSynchronize(void *s) { (void)s; return kOk; }
int hipMalloc(void **p, size_t bytes)
{
    ++calls;
    if (calls >= first_bad && calls <= last_bad) return kOutOfMemory;
    if (refuse_to && bytes >= refuse_from && bytes <= refuse_to) return kOutOfMemory;
    *p = calloc(1, bytes ? bytes : 1);
    if (!*p) return kOutOfMemory;
    ++live;
    return kOk;
}
int hipFree(void *p)
{
    if (p) --live;
    free(p);
    return kOk;
}
int hipHostMalloc(void **p, size_t bytes, unsigned flags) { (void)p; (void)bytes; (void)flags; return kOutOfMemory; }
int hipMemcpy(void *dst, const void *src, size_t bytes, int kind) { (void)kind; memcpy(dst, src, bytes); return kOk; }
int hipMemcpyAsync(void *dst, const void *src, size_t bytes, int kind, void *s)
{
    (void)kind;
    (void)s;
    memcpy(dst, src, bytes);
    return kOk;
}
int hipMemsetAsync(void *dst, int v, size_t bytes, void *s) { (void)s; memset(dst, v, bytes); return kOk; }
int hipLaunchKernel(const void *fn, ...) { (void)fn; return kOk; }
