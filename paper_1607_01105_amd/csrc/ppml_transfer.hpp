// ppml_transfer.hpp -- host side of the set and get calls: FP64 arrays of the
// caller's (pageable memory) to and from arrays of the storage type on the
// device.
//
// A pageable copy goes through the runtime's own staging at 11 GB/s, and one
// host thread checks or converts about as fast.  Here threads take chunks of
// the array in turn, each with two pinned buffers of its own: it checks, or
// converts, one chunk while the other is on the bus, and FP32 states cross the
// bus as FP32.  hipStreamPerThread names another stream in every thread, and
// only the caller's is ordered with the caller's steps: on that handle the
// caller's thread moves every chunk.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <exception>
#include <mutex>
#include <thread>
#include <vector>

#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
#include <xmmintrin.h>
#endif

namespace ppml {

// Bytes of a pinned buffer and most threads of a transfer.  128^3 FP32, six
// arrays of 16.8 MB set / got, ms: 256 KiB 8 threads 5.1 / 4.4, 512 KiB 8 3.6 /
// 3.2, 1 MiB 4 3.0 / 2.7, 1 MiB 8 3.0 / 3.1, 4 MiB 4 2.9 / 4.0 (through the
// runtime's staging 10.6 / 5.9).
constexpr size_t XFER_CHUNK = 1 << 20;
constexpr int XFER_THREADS = 4;
constexpr long long XFER_LEAST = 1 << 16; // values: fewer are converted faster than a thread starts
constexpr int CHECK_THREADS = 8;          // of a check, which waits for nothing but memory
constexpr size_t XFER_IDLE = 8;           // most idle lanes kept (2 MiB of pinned memory each)

// Two pinned buffers and the events of the copies that use them.
struct XferLane {
    int device = -1;
    void *buf[2] = {nullptr, nullptr};
    hipEvent_t ev[2] = {nullptr, nullptr};
    bool busy[2] = {false, false};
    bool lost = false;  // a copy may still use a buffer: the lane is not used or freed again

    hipError_t init(int dev)
    {
        hipError_t e = hipSuccess;
        for (int i = 0; i < 2 && e == hipSuccess; i++) e = hipHostMalloc(&buf[i], XFER_CHUNK, hipHostMallocPortable);
        return e == hipSuccess ? bind(dev) : e;
    }
    // The events belong to a device (the current one), the buffers to all.
    hipError_t bind(int dev)
    {
        hipError_t e = hipSuccess;
        for (int i = 0; i < 2 && e == hipSuccess; i++) {
            if (ev[i]) (void)hipEventDestroy(ev[i]);
            ev[i] = nullptr;
            e = hipEventCreateWithFlags(&ev[i], hipEventDisableTiming);
        }
        device = e == hipSuccess ? dev : -1;
        return e;
    }
    void free()
    {
        for (int i = 0; i < 2; i++) {
            if (ev[i]) (void)hipEventDestroy(ev[i]);
            if (buf[i]) (void)hipHostFree(buf[i]);
        }
    }
    // After a copy of buffer i on the stream: its event, or where that cannot be
    // recorded the copy's end.
    hipError_t mark(int i, hipStream_t stream)
    {
        const hipError_t e = hipEventRecord(ev[i], stream);
        busy[i] = e == hipSuccess;
        if (e != hipSuccess && hipStreamSynchronize(stream) != hipSuccess) lost = true;
        return e;
    }
    hipError_t wait(int i)
    {
        if (!busy[i]) return hipSuccess;
        busy[i] = false;
        return hipEventSynchronize(ev[i]);
    }
};

// Lanes no call is using, shared by every grid of the process: a call takes
// what it needs, one of its device if there is one, and gives it back; past
// XFER_IDLE they are freed.
class XferPool {
public:
    XferPool() { idle_.reserve(XFER_IDLE); }
    // (device: the current one)
    XferLane *take(int device, hipError_t &err)
    {
        XferLane *l = nullptr;
        {
            std::lock_guard<std::mutex> lock(mu_);
            size_t at = 0;
            while (at < idle_.size() && idle_[at]->device != device) at++;
            if (at == idle_.size()) at = 0;
            if (at < idle_.size()) {
                l = idle_[at];
                idle_.erase(idle_.begin() + (std::ptrdiff_t)at);
            }
        }
        if (l) {
            err = l->device == device ? hipSuccess : l->bind(device);
        } else {
            l = new XferLane;
            err = l->init(device);
        }
        if (err == hipSuccess) return l;
        l->free();
        delete l;
        return nullptr;
    }
    void give(XferLane *l)
    {
        if (l->lost) return;
        {
            std::lock_guard<std::mutex> lock(mu_);
            if (idle_.size() < XFER_IDLE) {
                idle_.push_back(l);
                return;
            }
        }
        l->free();
        delete l;
    }

private:
    std::mutex mu_;
    std::vector<XferLane *> idle_;
};
// (never destroyed: the runtime may already be gone when static objects are)
inline XferPool &xfer_pool()
{
    static XferPool *p = new XferPool;
    return *p;
}

// Runs f() on n threads, the caller's among them.
template <typename F> void on_threads(int n, F &&f)
{
    std::vector<std::thread> ts;
    try {
        ts.reserve((size_t)(n > 1 ? n - 1 : 0));
        for (int i = 1; i < n; i++) ts.emplace_back(f);
    } catch (const std::exception &) {
        // fewer threads: the others take the rest of the chunks
    }
    f();
    for (std::thread &t : ts) t.join();
}

// Keeps the caller's current device over a call.
struct XferDevice {
    int prev = -1;
    XferDevice()
    {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    }
    ~XferDevice()
    {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
};

// Most threads that may issue copies on the stream.
inline int xfer_most(hipStream_t stream) { return stream == hipStreamPerThread ? 1 : XFER_THREADS; }

inline int xfer_threads(size_t items, int most)
{
    const unsigned hw = std::thread::hardware_concurrency();
    return (int)std::min<size_t>(items, std::min<size_t>((size_t)most, hw > 0 ? hw : 1));
}

// Rounding of the host's checks and conversions, for the calling thread: to
// nearest, no exception trapped and no flag left, whatever the caller (whose
// settings its threads inherit) has set.  Conversions treat FP32 subnormals as
// the device does: the product build flushes them to zero, the exact build
// keeps them.
class XferRounding {
public:
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
#ifdef PPML_EXACT
    static constexpr unsigned FLUSH = 0;
#else
    static constexpr unsigned FLUSH = 0x8040;  // results to zero, subnormal operands read as zero
#endif
    explicit XferRounding(bool convert) : old_(_mm_getcsr()) { _mm_setcsr(0x1F80u | (convert ? FLUSH : 0u)); }
    ~XferRounding() { _mm_setcsr(old_); }

private:
    unsigned old_;
#else
    explicit XferRounding(bool) {}
#endif
};

// Host FP64 values to the storage type, and back.
template <typename T> void xfer_convert(const double *s, long long n, T *d)
{
    if (sizeof(T) == sizeof(double)) {
        std::memcpy(d, s, (size_t)n * sizeof(T));
        return;
    }
    const XferRounding mode(true);
    for (long long i = 0; i < n; i++) d[i] = (T)s[i];
}
inline void xfer_widen(const double *s, long long n, double *d) { std::memcpy(d, s, (size_t)n * sizeof(double)); }
inline void xfer_widen(const float *s, long long n, double *d)
{
    const XferRounding mode(true);
    for (long long i = 0; i < n; i++) d[i] = (double)s[i];
}

// Whether every value is finite (and, where asked, positive).
inline bool xfer_check(const double *a, long long n, bool positive)
{
    constexpr long long C = 1 << 17;
    const size_t items = (size_t)((n + C - 1) / C);
    std::atomic<size_t> next{0};
    std::atomic<bool> ok{true};
    on_threads(xfer_threads(items, CHECK_THREADS), [&] {
        for (size_t q; ok.load(std::memory_order_relaxed) && (q = next.fetch_add(1)) < items;) {
            const long long b = (long long)q * C, e = std::min(n, b + C);
            bool good = true;
            const XferRounding mode(false);
            if (positive)
                for (long long i = b; i < e; i++) good &= a[i] > 0.0 && a[i] <= 1.7976931348623157e308;
            else
                for (long long i = b; i < e; i++) good &= std::fabs(a[i]) <= 1.7976931348623157e308;
            if (!good) ok.store(false);
        }
    });
    return ok.load();
}

// The lanes of an upload whose copies may still be under way: they go back to
// the pool when the caller has waited for the stream, at the latest with this.
class XferHold {
public:
    ~XferHold() { (void)release(); }
    void keep(XferLane *l) { lanes_[n_.fetch_add(1)] = l; }
    hipError_t release()
    {
        hipError_t e = hipSuccess;
        for (int i = n_.exchange(0) - 1; i >= 0; i--) {
            for (int b = 0; b < 2; b++) {
                const hipError_t w = lanes_[i]->wait(b);
                if (e == hipSuccess) e = w;
            }
            xfer_pool().give(lanes_[i]);
        }
        return e;
    }

private:
    XferLane *lanes_[XFER_THREADS];
    std::atomic<int> n_{0};
};

// Host FP64 arrays src[0 .. nsrc), n values each (nullptr: zeros), to the device
// array dst of nsrc n values of type T, on the stream.  The host arrays have been
// read when the call returns; the copies end in the stream's order, and the
// buffers they come from are held until then (waiting for them here cost a set
// call of 64 cells 10 of its 75 us).
template <typename T>
hipError_t xfer_upload(int device, hipStream_t stream, const double *const *src, int nsrc, long long n, T *dst,
                       XferHold &hold)
{
    // chunks of the buffers' size, or smaller ones down to XFER_LEAST values
    // so that every thread has one to convert (256^2 FP32 primitives 0.34 ms
    // instead of 0.40); small arrays by the caller's thread alone
    long long there = 0;
    for (int f = 0; f < nsrc; f++) there += src[f] ? n : 0;
    const long long C = std::min<long long>(XFER_CHUNK / sizeof(T),
                                            std::max<long long>(XFER_LEAST, (there + XFER_THREADS - 1) / XFER_THREADS));
    // runs of arrays that are there, as ranges of dst
    long long beg_of[8], end_of[8];
    size_t first[9] = {0};  // the runs' first chunks
    int runs = 0;
    for (int f = 0; f < nsrc;) {
        int e = f;
        while (e < nsrc && (src[e] != nullptr) == (src[f] != nullptr)) e++;
        if (src[f]) {
            beg_of[runs] = f * n;
            end_of[runs] = e * n;
            first[runs + 1] = first[runs] + (size_t)((end_of[runs] - beg_of[runs] + C - 1) / C);
            runs++;
        } else {
            const hipError_t z = hipMemsetAsync(dst + f * n, 0, (size_t)((e - f) * n) * sizeof(T), stream);
            if (z != hipSuccess) return z;
        }
        f = e;
    }
    const size_t items = first[runs];
    std::atomic<size_t> next{0};
    std::atomic<int> err{(int)hipSuccess};
    const XferDevice keep;
    on_threads(xfer_threads(std::min<size_t>(items, 1 + (size_t)(there / XFER_LEAST)), xfer_most(stream)), [&] {
        hipError_t e = hipSetDevice(device);
        XferLane *l = nullptr;
        if (e == hipSuccess) {
            try {
                l = xfer_pool().take(device, e);
            } catch (const std::exception &) {
                e = hipErrorOutOfMemory;
            }
        }
        int b = 0;
        size_t q;
        while (l && e == hipSuccess && err.load() == (int)hipSuccess && (q = next.fetch_add(1)) < items) {
            int run = 0;
            while (q >= first[run + 1]) run++;
            const long long beg = beg_of[run] + (long long)(q - first[run]) * C, end = std::min(end_of[run], beg + C);
            if ((e = l->wait(b)) != hipSuccess) break;
            T *p = (T *)l->buf[b];
            for (long long i = beg; i < end;) {
                const long long f = i / n, lo = i - f * n, m = std::min(end - i, n - lo);
                xfer_convert(src[f] + lo, m, p);
                p += m;
                i += m;
            }
            e = hipMemcpyAsync(dst + beg, l->buf[b], (size_t)(end - beg) * sizeof(T), hipMemcpyHostToDevice, stream);
            if (e == hipSuccess) e = l->mark(b, stream);
            b ^= 1;
        }
        if (l) hold.keep(l);
        if (e != hipSuccess) err.store((int)e);
    });
    return (hipError_t)err.load();
}

// The device array src of n values of type T, after the stream's work, to the
// host FP64 array dst; complete when the call returns.
template <typename T>
hipError_t xfer_download(int device, hipStream_t stream, const T *src, long long n, double *dst)
{
    constexpr long long C = XFER_CHUNK / sizeof(T);
    const size_t items = (size_t)((n + C - 1) / C);
    std::atomic<size_t> next{0};
    std::atomic<int> err{(int)hipSuccess};
    const XferDevice keep;
    on_threads(xfer_threads(items, xfer_most(stream)), [&] {
        hipError_t e = hipSetDevice(device);
        XferLane *l = nullptr;
        if (e == hipSuccess) {
            try {
                l = xfer_pool().take(device, e);
            } catch (const std::exception &) {
                e = hipErrorOutOfMemory;
            }
        }
        size_t at[2] = {0, 0};
        auto fetch = [&](int b) {
            if (err.load() != (int)hipSuccess || (at[b] = next.fetch_add(1)) >= items) return false;
            const long long beg = (long long)at[b] * C, m = std::min(n - beg, C);
            e = hipMemcpyAsync(l->buf[b], src + beg, (size_t)m * sizeof(T), hipMemcpyDeviceToHost, stream);
            if (e == hipSuccess) e = l->mark(b, stream);
            return e == hipSuccess;
        };
        int b = 0;
        bool have = l && e == hipSuccess && fetch(0);
        while (have) {
            const bool more = fetch(b ^ 1);
            const hipError_t w = l->wait(b);
            if (w != hipSuccess) {
                e = w;
                break;
            }
            const long long beg = (long long)at[b] * C, m = std::min(n - beg, C);
            xfer_widen((const T *)l->buf[b], m, dst + beg);
            b ^= 1;
            have = more;
        }
        if (l) {
            for (int i = 0; i < 2; i++) (void)l->wait(i);
            xfer_pool().give(l);
        }
        if (e != hipSuccess) err.store((int)e);
    });
    return (hipError_t)err.load();
}

}  // namespace ppml
