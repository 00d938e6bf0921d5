// A device of host memory for the CPU tests of the library's host code: the HIP calls it makes, with
// allocations that can be made to fail, on the device and (operator new) on the host.  Kernels do not run
// (but for the one that brings results to the host), so only what happens before the first result of one is
// read can be tested, and what follows a result that a test supplies (fake_hip_answer).
#include <cstdlib>
#include <cstring>
#include <new>

static int new_calls, bad_new; // the bad_new-th from now on throws, counted from 1; 0: none
void *operator new(std::size_t bytes)
{
    if (bad_new && ++new_calls == bad_new) throw std::bad_alloc();
    if (void *p = std::malloc(bytes ? bytes : 1)) return p;
    throw std::bad_alloc();
}
void *operator new(std::size_t bytes, const std::nothrow_t &) noexcept
{
    if (bad_new && ++new_calls == bad_new) return nullptr;
    return std::malloc(bytes ? bytes : 1);
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

extern "C" {
enum { kOk = 0, kOutOfMemory = 2, kLaunchFailure = 719, kCaptureImplicit = 906 };
static int calls, first_bad, last_bad; // allocations [first_bad, last_bad] fail, counted from 1
static std::size_t refuse_from, refuse_to; // and those of refuse_from to refuse_to bytes, so often
static int refuse_left;
static long live;

void fake_hip_fail(int first, int last)
{
    calls = 0;
    first_bad = first;
    last_bad = last;
}
void fake_hip_refuse(std::size_t from, std::size_t to)
{
    refuse_from = from;
    refuse_to = to;
    refuse_left = 1 << 30;
}
void fake_hip_refuse_times(int times) { refuse_left = times; }
void fake_new_fail(int at)
{
    new_calls = 0;
    bad_new = at;
}
int fake_new_calls(void) { return new_calls; }
int fake_hip_allocations(void) { return calls; }
long fake_hip_live(void) { return live; }

static std::size_t free_bytes = 100, total_bytes = 100;
static int capturing;
void fake_hip_memory(std::size_t free_now, std::size_t total) { free_bytes = free_now; total_bytes = total; }
void fake_hip_capture(int on) { capturing = on; }

int hipMemGetInfo(std::size_t *f, std::size_t *t) { *f = free_bytes; *t = total_bytes; return kOk; }
int hipStreamIsCapturing(void *s, int *status) { (void)s; *status = capturing; return kOk; }
int hipThreadExchangeStreamCaptureMode(int *mode) { (void)mode; return kOk; }
int hipGetDeviceCount(int *n) { *n = 1; return kOk; }
int hipGetDevice(int *d) { *d = 0; return kOk; }
int hipSetDevice(int d) { (void)d; return kOk; }
int hipGetLastError(void) { return kOk; }
int hipDeviceSynchronize(void) { return kOk; }
int hipMalloc(void **p, std::size_t bytes)
{
    ++calls;
    if (calls >= first_bad && calls <= last_bad) return kOutOfMemory;
    if (refuse_to && bytes >= refuse_from && bytes <= refuse_to && refuse_left > 0) {
        --refuse_left;
        return kOutOfMemory;
    }
    *p = std::calloc(1, bytes ? bytes : 1);
    if (!*p) return kOutOfMemory;
    ++live;
    return kOk;
}
int hipFree(void *p)
{
    if (p) --live;
    std::free(p);
    return kOk;
}
// Streams: none unless asked for, and then all the same.
static int streams, streams_made;
void fake_hip_streams(int on) { streams = on; }
int fake_hip_streams_made(void) { return streams_made; }
int hipStreamCreateWithFlags(void **s, unsigned flags)
{
    (void)flags;
    static int made;
    if (!streams) return kOutOfMemory;
    ++streams_made;
    *s = &made;
    return kOk;
}
int hipStreamDestroy(void *s) { (void)s; return kOk; }
int hipGetStreamDeviceId(void *s) { (void)s; return 0; }
int hipFuncSetAttribute(const void *fn, int attribute, int value) { (void)fn, (void)attribute, (void)value; return kOk; }
int hipDeviceGetAttribute(int *value, int attribute, int device) { (void)attribute, (void)device; *value = 256; return kOk; }
int hipGetDevicePropertiesR0600(void *properties, int device)
{
    (void)device;
    std::memset(properties, 0, 1472); // hipDeviceProp_t
    return kOk;
}
// Pinned memory: none unless asked for.
static int pinned;
static unsigned pinned_flags = ~0u; // those that all of it was asked for with
void fake_hip_pinned(int on) { pinned = on; }
unsigned fake_hip_pinned_flags(void) { return pinned_flags; }
int hipHostMalloc(void **p, std::size_t bytes, unsigned flags)
{
    if (!pinned) return kOutOfMemory;
    pinned_flags &= flags;
    *p = std::calloc(1, bytes);
    return *p ? kOk : kOutOfMemory;
}
// A copy of `bytes` bytes to the host brings these in place of what is there (bytes 0: none does).
static std::size_t answer_bytes[4];
static unsigned char answers[4][128];
void fake_hip_answer(int slot, std::size_t bytes, const void *what)
{
    answer_bytes[slot] = bytes;
    std::memcpy(answers[slot], what, bytes);
}
static void to_host(void *dst, const void *src, std::size_t bytes)
{
    std::memcpy(dst, src, bytes);
    for (int i = 0; i < 4; ++i)
        if (bytes && bytes == answer_bytes[i]) std::memcpy(dst, answers[i], bytes);
}
int hipMemcpy(void *dst, const void *src, std::size_t bytes, int kind)
{
    if (capturing) return kCaptureImplicit;
    kind == 2 ? to_host(dst, src, bytes) : (void)std::memcpy(dst, src, bytes);
    return kOk;
}
int hipMemcpyAsync(void *dst, const void *src, std::size_t bytes, int kind, void *s)
{
    (void)s;
    kind == 2 ? to_host(dst, src, bytes) : (void)std::memcpy(dst, src, bytes);
    return kOk;
}
int hipMemsetAsync(void *dst, int v, std::size_t bytes, void *s) { (void)s; std::memset(dst, v, bytes); return kOk; }
static int launches;
int fake_hip_launches(void) { return launches; }
struct Dim3 { unsigned x, y, z; };
static thread_local struct { Dim3 grid, block; std::size_t lds; void *stream; } pushed; // by the caller of a kernel, for its stub
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, std::size_t lds, void *stream)
{
    pushed = {grid, block, lds, stream};
    return kOk;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, std::size_t *lds, void **stream)
{
    *grid = pushed.grid;
    *block = pushed.block;
    *lds = pushed.lds;
    *stream = pushed.stream;
    return kOk;
}
// The one kernel that is run: deliver_kernel, which leaves results in pinned memory.  Its next run can be kept back: the wait for it
// fails, and it runs when the next one would, which then does so when it is waited for.
static const void *deliver_kernel;
void __hipRegisterFunction(void *, const void *fn, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    if (std::strstr(name, "deliver_kernel")) deliver_kernel = fn;
}
struct Delivery {
    void *to;
    unsigned char what[256];
    std::size_t bytes;
    unsigned *flag, seq;
};
static Delivery kept;
static enum { kRuns, kNextKept, kKept, kLate } delivery = kRuns;
void fake_hip_keep_back(void) { delivery = kNextKept; }
static void arrive(const Delivery &d)
{
    std::memcpy(d.to, d.what, d.bytes);
    __atomic_store_n(d.flag, d.seq, __ATOMIC_RELEASE);
}
static void deliver(void **args)
{
    Delivery d = {*(void **)args[0], {}, 4u * (std::size_t)*(int *)args[2], *(unsigned **)args[3], *(unsigned *)args[4]};
    to_host(d.what, *(const void **)args[1], d.bytes);
    if (delivery == kRuns) return arrive(d);
    if (delivery == kKept) arrive(kept);
    kept = d;
    delivery = delivery == kKept ? kLate : kKept;
}
int hipStreamSynchronize(void *s)
{
    (void)s;
    if (delivery == kKept) return kLaunchFailure;
    if (delivery == kLate) arrive(kept), delivery = kRuns;
    return kOk;
}
int hipLaunchKernel(const void *fn, Dim3 grid, Dim3 block, void **args, std::size_t lds, void *stream)
{
    (void)grid, (void)block, (void)lds, (void)stream;
    ++launches;
    if (fn == deliver_kernel) deliver(args);
    return kOk;
}
}
