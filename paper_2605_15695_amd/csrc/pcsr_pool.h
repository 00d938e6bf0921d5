// Device memory of the library: handles, workspaces and the scratch of the set-up calls come
// from a cache of freed blocks, one per GPU.  A build needs some twenty arrays; released with
// hipFree they cost 2-5 ms per build of a 16 M-nonzero graph (each large hipFree unmaps its
// pages and waits for the device), a third of building, multiplying and releasing it.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <mutex>
#include <thread>

namespace pcsr {

// Blocks kept for reuse per GPU at most; beyond it the longest unused go back to the driver, and
// so does a block that kPoolIdleAllocs allocations have passed over.  All of them go back
// before an allocation is reported as out of memory, when the caller asks (pcsr_release_cached), and
// when torch asks the driver for more with less than one part in kPoolLowMemory of the device free.
constexpr size_t kPoolBytes = size_t(1) << 30;
constexpr uint64_t kPoolIdleAllocs = 1024;
constexpr size_t kPoolLowMemory = 8;

// On the current device.  Thread safe.  Contents are undefined.
hipError_t pool_alloc(void **p, size_t bytes) noexcept;
// No work that uses the block may be running or enqueued: the caller has waited for the device
// (pool_quiesce) or for the stream that used it.  nullptr is a no-op.
void pool_free(void *p) noexcept;
// Waits for a device, as hipFree would.  false: that failed (a stream capture in progress, say)
// and the blocks have to go back through pool_release instead.
bool pool_quiesce(int device);
void pool_release(void *p) noexcept; // hipFree, past the cache
// Gives the blocks kept for the current device back to the driver; bytes: how many that were.
hipError_t pool_give_back(size_t *bytes);

// Large synchronous copies between pageable host memory and the current device.  A few threads
// each move 1 MB pieces through pinned buffers of their own (kept for reuse, 16 MB in all), so
// that faulting in, copying and transfer overlap: hipMemcpy writes a fresh 96 MB host array at
// 4 GB/s (the page faults are taken one by one) and reads one at 30 GB/s; this way it is 20-30
// and 45 GB/s.  One call at a time uses the threads, others meanwhile take hipMemcpy.
// Below kStagedBytes: hipMemcpy.
constexpr size_t kStagedBytes = size_t(4) << 20;
hipError_t copy_to_host(void *dst, const void *src, size_t bytes);
hipError_t copy_to_device(void *dst, const void *src, size_t bytes);

// Where the set-up code enqueues its work: the null stream, or, on a thread that has put a SetupOn in scope, the stream of that.
hipStream_t setup_stream() noexcept;
// hipMemcpy there.  What a few kernels have counted is brought to pinned memory by one more, with a flag after it that the host looks
// for: 9.3 us from the launch of the last of them where hipMemcpy takes 14.5, and 23 on another stream than the null stream.
hipError_t setup_copy(void *dst, const void *src, size_t bytes, hipMemcpyKind kind) noexcept;
// Waits for what this thread has enqueued there, unless setup_copy has and nothing was since (setup_stream was not asked for).
hipError_t setup_wait() noexcept;
class SetupOn {
public:
    explicit SetupOn(hipStream_t s) noexcept;
    SetupOn(const SetupOn &) = delete;
    SetupOn &operator=(const SetupOn &) = delete;
    ~SetupOn();

private:
    hipStream_t before;
};
// The current device's stream for set-up work beside that on the null stream, which it does not wait for, nor that for it: what it is
// to read has to be there.  One caller at a time has it; others, and one for whom none could be made, get null.
class SideStream {
public:
    SideStream() noexcept;
    SideStream(const SideStream &) = delete;
    SideStream &operator=(const SideStream &) = delete;
    ~SideStream();
    hipStream_t get() const noexcept { return stream; }

private:
    hipStream_t stream = nullptr;
    int device = -1;
};

// Values that come later than the pattern they belong to.  wait(): until they are there, for what is enqueued on
// setup_stream() afterwards.
class Late {
public:
    virtual hipError_t wait() noexcept = 0;

protected:
    ~Late() = default;
};

// copy_to_device beside what the caller does meanwhile, on threads (half as many) and pinned buffers of its own.
// Nothing enqueued may still use dst; src has to stay until wait() (or the destructor) returns.  Where no thread is to be had the
// copy is made by start().
// wait() may be called by several threads.
class Upload final : public Late {
public:
    Upload() = default;
    Upload(const Upload &) = delete;
    Upload &operator=(const Upload &) = delete;
    ~Upload() { (void)wait(); }
    void start(void *dst, const void *src, size_t bytes) noexcept;
    hipError_t wait() noexcept override;
    bool beside() const noexcept { return on_thread; } // whether start() left the copy to a thread

private:
    std::mutex joining;
    std::thread thread;
    bool on_thread = false;
    hipError_t result = hipSuccess;
};

} // namespace pcsr

// For torch's allocator, which asks before it takes more memory from the driver (pcsr_py.cpp):
// pcsr_release_cached if the device is that low and `stream` is not being captured.  Returns the
// bytes given back.
extern "C" int64_t pcsr_release_cached_if_low(void *stream);
