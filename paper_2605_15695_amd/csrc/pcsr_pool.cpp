#include "pcsr_pool.h"
#include "pcsr_build_gpu.h"

#include <algorithm>
#include <atomic>
#include <cstring>
#include <map>
#include <mutex>
#include <thread>
#include <unordered_map>
#include <vector>

namespace pcsr {
namespace {

struct Block {
    size_t bytes;
    int device;
};
struct Idle {
    void *p;
    uint64_t since; // allocation count when it was freed
};
struct Cache {
    std::multimap<size_t, Idle> idle; // by size
    size_t bytes = 0;
};

struct Pool {
    std::mutex mu;
    std::unordered_map<void *, Block> live;
    std::map<int, Cache> caches;
    uint64_t clock = 0;
};

Pool &pool()
{
    static Pool *p = new Pool; // never destroyed: handles may outlive static destruction
    return *p;
}

size_t rounded(size_t bytes)
{
    const size_t unit = bytes >= (size_t(1) << 20) ? size_t(1) << 20 : 4096;
    return (std::max<size_t>(bytes, 1) + unit - 1) / unit * unit;
}

void drop(Cache &c, std::multimap<size_t, Idle>::iterator it)
{
    (void)hipFree(it->second.p);
    c.bytes -= it->first;
    c.idle.erase(it);
}

} // namespace

hipError_t pool_alloc(void **out, size_t bytes) noexcept
try {
    *out = nullptr;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const size_t need = rounded(bytes);
    Pool &P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    ++P.clock;
    Cache &c = P.caches[dev];
    // a block up to a quarter (or 1 MB) larger than asked for
    auto it = c.idle.lower_bound(need);
    if (it != c.idle.end() && it->first <= need + std::max(need / 4, size_t(1) << 20)) {
        P.live[it->second.p] = {it->first, dev};
        *out = it->second.p;
        c.bytes -= it->first;
        c.idle.erase(it);
        return hipSuccess;
    }
    e = hipMalloc(out, need);
    if (e == hipErrorOutOfMemory && !c.idle.empty()) {
        (void)hipGetLastError();
        while (!c.idle.empty()) drop(c, c.idle.begin());
        e = hipMalloc(out, need);
    }
    if (e != hipSuccess) {
        *out = nullptr;
        return e;
    }
    P.live[*out] = {need, dev};
    return hipSuccess;
} catch (...) { // no host memory for the books
    if (*out) (void)hipFree(*out);
    *out = nullptr;
    return hipErrorOutOfMemory;
}

void pool_free(void *p) noexcept
{
    if (!p) return;
    Pool &P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    auto it = P.live.find(p);
    if (it == P.live.end()) {
        (void)hipFree(p);
        return;
    }
    Cache &c = P.caches[it->second.device];
    const size_t bytes = it->second.bytes;
    P.live.erase(it);
    if (bytes > kPoolBytes) {
        (void)hipFree(p);
        return;
    }
    try {
        c.idle.insert({bytes, {p, P.clock}});
    } catch (...) {
        (void)hipFree(p);
        return;
    }
    c.bytes += bytes;
    for (auto i = c.idle.begin(); i != c.idle.end();) {
        auto at = i++;
        if (P.clock - at->second.since > kPoolIdleAllocs) drop(c, at);
    }
    while (c.bytes > kPoolBytes) {
        auto oldest = c.idle.begin();
        for (auto i = c.idle.begin(); i != c.idle.end(); ++i)
            if (i->second.since < oldest->second.since) oldest = i;
        drop(c, oldest);
    }
}

bool pool_quiesce(int device)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    if (dev != device && hipSetDevice(device) != hipSuccess) return false;
    const hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) (void)hipGetLastError();
    if (dev != device) (void)hipSetDevice(dev);
    return e == hipSuccess;
}

void pool_release(void *p) noexcept
{
    if (!p) return;
    Pool &P = pool();
    {
        std::lock_guard<std::mutex> lock(P.mu);
        P.live.erase(p);
    }
    (void)hipFree(p);
}

hipError_t pool_give_back(size_t *bytes)
{
    *bytes = 0;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    // a capture that another thread has under way must not be ended by these frees: the blocks are no part of it
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    {
        Pool &P = pool();
        std::lock_guard<std::mutex> lock(P.mu);
        auto at = P.caches.find(dev);
        if (at != P.caches.end()) {
            *bytes = at->second.bytes;
            while (!at->second.idle.empty()) drop(at->second, at->second.idle.begin());
        }
    }
    if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
    return hipSuccess;
}

namespace {

constexpr int kCopyThreads = 8, kBesideThreads = 4;
constexpr size_t kPiece = size_t(1) << 20;

struct Lane { // one copying thread's buffers and stream
    char *pin[2] = {nullptr, nullptr};
    hipStream_t stream[2] = {nullptr, nullptr};
};
struct Lanes {
    std::mutex mu;
    std::map<int, std::vector<Lane>> per_device;
};
Lanes &lanes(bool beside) // of copies the caller waits for, of those beside its work
{
    static Lanes *l = new Lanes[2];
    return l[beside];
}

// The lanes of a device, made on first use; empty if that failed.  Lanes::mu held.
std::vector<Lane> &lanes_of(Lanes &all, int dev, int threads)
{
    std::vector<Lane> &v = all.per_device[dev];
    if (!v.empty()) return v;
    std::vector<Lane> made(threads);
    bool ok = true;
    for (Lane &l : made)
        for (int b = 0; b < 2 && ok; ++b)
            ok = hipHostMalloc((void **)&l.pin[b], kPiece, hipHostMallocDefault) == hipSuccess &&
                 hipStreamCreateWithFlags(&l.stream[b], hipStreamNonBlocking) == hipSuccess;
    if (ok) {
        v.swap(made);
    } else {
        (void)hipGetLastError();
        for (Lane &l : made)
            for (int b = 0; b < 2; ++b) {
                if (l.stream[b]) (void)hipStreamDestroy(l.stream[b]);
                if (l.pin[b]) (void)hipHostFree(l.pin[b]);
            }
    }
    return v;
}

hipError_t staged(char *dst, const char *src, size_t bytes, bool to_host, bool beside = false)
{
    const hipMemcpyKind kind = to_host ? hipMemcpyDeviceToHost : hipMemcpyHostToDevice;
    int dev = -1;
    if (bytes < kStagedBytes || hipGetDevice(&dev) != hipSuccess) return hipMemcpy(dst, src, bytes, kind);
    Lanes &all = lanes(beside);
    std::unique_lock<std::mutex> lock(all.mu, std::try_to_lock);
    if (!lock.owns_lock()) return hipMemcpy(dst, src, bytes, kind);
    const int threads = beside ? kBesideThreads : kCopyThreads;
    Lane *ls = nullptr;
    try {
        std::vector<Lane> &v = lanes_of(all, dev, threads);
        if (!v.empty()) ls = v.data();
    } catch (...) {
    }
    if (!ls) return hipMemcpy(dst, src, bytes, kind);
    // like hipMemcpy, after everything enqueued on the null stream
    hipError_t e = beside ? hipSuccess : hipStreamSynchronize(nullptr);
    if (e != hipSuccess) return e;
    std::atomic<int> failed{hipSuccess};
    const size_t pieces = (bytes + kPiece - 1) / kPiece;
    auto work = [&](int t) {
        Lane &l = ls[t];
        hipError_t r = hipSetDevice(dev);
        size_t wait[2] = {pieces, pieces}; // piece in flight in each buffer
        int b = 0;
        auto size = [&](size_t p) { return std::min(kPiece, bytes - p * kPiece); };
        auto settle = [&](int k) { // finishes what buffer k has in flight
            if (wait[k] == pieces) return;
            const hipError_t w = hipStreamSynchronize(l.stream[k]);
            if (w != hipSuccess) r = w;
            if (to_host && w == hipSuccess) std::memcpy(dst + wait[k] * kPiece, l.pin[k], size(wait[k]));
            wait[k] = pieces;
        };
        for (size_t p = t; p < pieces && r == hipSuccess; p += threads, b ^= 1) {
            settle(b);
            if (r != hipSuccess) break;
            const size_t at = p * kPiece;
            if (to_host) {
                r = hipMemcpyAsync(l.pin[b], src + at, size(p), kind, l.stream[b]);
            } else {
                std::memcpy(l.pin[b], src + at, size(p));
                r = hipMemcpyAsync(dst + at, l.pin[b], size(p), kind, l.stream[b]);
            }
            if (r == hipSuccess) wait[b] = p;
        }
        settle(b); // the older piece first
        settle(b ^ 1);
        if (r != hipSuccess) failed = r;
    };
    std::vector<std::thread> th;
    const int n = (int)std::min<size_t>(threads, pieces);
    try {
        for (int t = 1; t < n; ++t) th.emplace_back(work, t);
    } catch (...) { // no more threads: what they would have moved is moved here
    }
    const int started = (int)th.size() + 1;
    work(0);
    for (int t = started; t < n; ++t) work(t);
    for (std::thread &t : th) t.join();
    return (hipError_t)failed.load();
}

} // namespace

hipError_t copy_to_host(void *dst, const void *src, size_t bytes)
{
    return staged(static_cast<char *>(dst), static_cast<const char *>(src), bytes, true);
}

hipError_t copy_to_device(void *dst, const void *src, size_t bytes)
{
    return staged(static_cast<char *>(dst), static_cast<const char *>(src), bytes, false);
}

void Upload::start(void *dst, const void *src, size_t bytes) noexcept
{
    result = wait();
    on_thread = false;
    if (result != hipSuccess || bytes == 0) return;
    int dev = -1;
    if (bytes >= kStagedBytes && hipGetDevice(&dev) == hipSuccess) {
        try {
            thread = std::thread([=] {
                result = hipSetDevice(dev);
                if (result == hipSuccess)
                    result = staged(static_cast<char *>(dst), static_cast<const char *>(src), bytes, false, true);
            });
            on_thread = true;
            return;
        } catch (...) { // no thread
        }
    }
    result = copy_to_device(dst, src, bytes);
}

hipError_t Upload::wait() noexcept
{
    std::lock_guard<std::mutex> lock(joining);
    if (thread.joinable()) thread.join();
    return result;
}

namespace {
thread_local hipStream_t t_setup_stream = nullptr;

struct Side {
    hipStream_t stream = nullptr;
    bool taken = false;
};
struct Sides {
    std::mutex mu;
    std::map<int, Side> per_device;
};
Sides &sides()
{
    static Sides *s = new Sides;
    return *s;
}
} // namespace

namespace {
// Pinned memory that a kernel leaves results in for the host: of one thread at a time, kept for the next one when that ends.
// Coherent: the host looks at it while the kernel is still there.
constexpr size_t kMailBytes = 256;
struct Mail {
    unsigned char data[kMailBytes];
    unsigned seq; // of the results in it
};
struct Box {
    Mail *mail = nullptr;
    unsigned last = 0; // number of the last hand-over, whether it arrived or not
};
struct BoxList {
    std::mutex mu;
    std::vector<Box> idle;
};
BoxList &box_list()
{
    static BoxList *l = new BoxList;
    return *l;
}
struct OwnBox {
    Box box;
    bool tried = false;
    Box *get() noexcept
    try {
        if (box.mail) return &box;
        if (tried) return nullptr;
        tried = true;
        BoxList &l = box_list();
        {
            std::lock_guard<std::mutex> lock(l.mu);
            l.idle.reserve(l.idle.size() + 1);
            if (!l.idle.empty()) {
                box = l.idle.back();
                l.idle.pop_back();
                return &box;
            }
        }
        void *p = nullptr;
        if (hipHostMalloc(&p, sizeof(Mail), hipHostMallocPortable | hipHostMallocCoherent) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        box.mail = static_cast<Mail *>(p);
        box.mail->seq = box.last;
        return &box;
    } catch (...) {
        return nullptr;
    }
    // What was to arrive may do so at any time: never used again, nor given back.
    void retire() noexcept
    {
        box = Box();
        tried = false;
    }
    ~OwnBox()
    {
        if (!box.mail) return;
        try {
            BoxList &l = box_list();
            std::lock_guard<std::mutex> lock(l.mu);
            l.idle.push_back(box);
        } catch (...) {
        }
    }
};
thread_local OwnBox t_box;
thread_local bool t_enqueued = true; // on t_setup_stream, since it was last known to be idle
constexpr int kSpins = 200000;       // some milliseconds; then the runtime's own wait, which also reports errors
} // namespace

hipStream_t setup_stream() noexcept
{
    t_enqueued = true;
    return t_setup_stream;
}

hipError_t setup_wait() noexcept
{
    if (!t_enqueued) return hipSuccess;
    const hipError_t e = hipStreamSynchronize(t_setup_stream);
    if (e == hipSuccess) t_enqueued = false;
    return e;
}

hipError_t setup_copy(void *dst, const void *src, size_t bytes, hipMemcpyKind kind) noexcept
{
    const hipStream_t s = t_setup_stream;
    Box *const box = kind == hipMemcpyDeviceToHost && bytes <= kMailBytes && bytes % 4 == 0 ? t_box.get() : nullptr;
    if (box) {
        Mail *const mail = box->mail;
        const unsigned seq = ++box->last;
        hipError_t e = deliver(mail->data, src, (int)(bytes / 4), &mail->seq, seq, s);
        if (e != hipSuccess) {
            t_box.retire();
            return e;
        }
        auto arrived = [&] { return __atomic_load_n(&mail->seq, __ATOMIC_ACQUIRE) == seq; };
        // A copy on the null stream is refused while some stream is being captured, even one of nothing; kernels are not, and
        // would count what the capture is yet to make.  (0.6 us, while the kernel runs.)
        if (!s) e = hipMemcpy(dst, src, 0, kind);
        for (int i = 0; e == hipSuccess && i < kSpins && !arrived(); ++i) __builtin_ia32_pause();
        if (!arrived()) {
            const hipError_t w = hipStreamSynchronize(s);
            if (e == hipSuccess) e = w;
            if (!arrived()) {
                t_box.retire();
                if (e == hipSuccess) e = hipErrorUnknown;
            }
        }
        if (e != hipSuccess) return e;
        std::memcpy(dst, mail->data, bytes);
        t_enqueued = false;
        return hipSuccess;
    }
    if (!s) {
        const hipError_t e = hipMemcpy(dst, src, bytes, kind);
        if (e == hipSuccess && kind == hipMemcpyDeviceToHost) t_enqueued = false;
        return e;
    }
    const hipError_t e = hipMemcpyAsync(dst, src, bytes, kind, s), w = hipStreamSynchronize(s);
    return e != hipSuccess ? e : w;
}

SetupOn::SetupOn(hipStream_t s) noexcept : before(t_setup_stream)
{
    t_setup_stream = s;
    t_enqueued = true;
}
SetupOn::~SetupOn()
{
    t_setup_stream = before;
    t_enqueued = true;
}

SideStream::SideStream() noexcept
try {
    if (hipGetDevice(&device) != hipSuccess) return;
    Sides &all = sides();
    std::lock_guard<std::mutex> lock(all.mu);
    Side &s = all.per_device[device];
    if (s.taken) return;
    if (!s.stream && hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking) != hipSuccess) {
        (void)hipGetLastError();
        s.stream = nullptr;
        return;
    }
    s.taken = true;
    stream = s.stream;
} catch (...) { // no host memory for the books
}

SideStream::~SideStream()
{
    if (!stream) return;
    Sides &all = sides();
    std::lock_guard<std::mutex> lock(all.mu);
    all.per_device[device].taken = false;
}

} // namespace pcsr

extern "C" int64_t pcsr_release_cached_if_low(void *stream)
{
    size_t free = 0, total = 0, bytes = 0;
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    const bool idle = hipStreamIsCapturing(static_cast<hipStream_t>(stream), &status) == hipSuccess &&
                      status == hipStreamCaptureStatusNone;
    const bool low = idle && hipMemGetInfo(&free, &total) == hipSuccess && free < total / pcsr::kPoolLowMemory;
    if (!idle || (low && pcsr::pool_give_back(&bytes) != hipSuccess)) (void)hipGetLastError();
    return (int64_t)bytes;
}
