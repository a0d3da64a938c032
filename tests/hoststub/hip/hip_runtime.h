// Stand-in for the HIP runtime calls of ppml_transfer.hpp, for its CPU tests.
// A copy or an event is an entry of its stream's queue and takes effect only
// when the stream or an event behind it is waited for, so that a buffer used
// again too early shows in the data.  A call can be made to fail.
#pragma once

#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <mutex>
#include <thread>
#include <utility>
#include <vector>

enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2, hipErrorUnknown = 999 };
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost };
constexpr unsigned hipHostMallocPortable = 1, hipEventDisableTiming = 2;
typedef struct stub_stream *hipStream_t;
#define hipStreamPerThread ((hipStream_t)2)

struct stub_event {
    int device;
    bool pending = false;
};
typedef stub_event *hipEvent_t;

struct stub_op {
    void *dst = nullptr;
    const void *src = nullptr;
    size_t bytes = 0;  // of a copy; src null: zeros
    hipEvent_t event = nullptr;
};

struct stub_runtime {
    std::mutex mu;
    typedef std::pair<hipStream_t, std::thread::id> Key;  // a per-thread stream is one per thread
    std::map<Key, std::deque<stub_op>> queue;
    std::vector<std::thread::id> copied_by;  // thread of every copy
    int records = 0, fail_record = -1;       // event records so far, the one that fails
    int host_allocs = 0, event_mismatches = 0;
    std::map<std::thread::id, int> device;

    static Key key(hipStream_t s) { return {s, s == hipStreamPerThread ? std::this_thread::get_id() : std::thread::id()}; }
    static void run(std::deque<stub_op> &q, hipEvent_t until)
    {
        while (!q.empty()) {
            const stub_op op = q.front();
            q.pop_front();
            if (op.src) std::memcpy(op.dst, op.src, op.bytes);
            else if (op.dst) std::memset(op.dst, 0, op.bytes);
            if (op.event) op.event->pending = false;
            if (op.event && op.event == until) return;
        }
    }
};
inline stub_runtime &stub()
{
    static stub_runtime r;
    return r;
}

inline hipError_t hipGetDevice(int *d)
{
    std::lock_guard<std::mutex> l(stub().mu);
    *d = stub().device[std::this_thread::get_id()];
    return hipSuccess;
}
inline hipError_t hipSetDevice(int d)
{
    std::lock_guard<std::mutex> l(stub().mu);
    stub().device[std::this_thread::get_id()] = d;
    return hipSuccess;
}
inline hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    std::lock_guard<std::mutex> l(stub().mu);
    stub().host_allocs++;
    *p = std::malloc(n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
inline hipError_t hipHostFree(void *p)
{
    std::free(p);
    return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    std::lock_guard<std::mutex> l(stub().mu);
    *e = new stub_event{stub().device[std::this_thread::get_id()]};
    return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e)
{
    delete e;
    return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    std::lock_guard<std::mutex> l(stub().mu);
    if (stub().records++ == stub().fail_record) return hipErrorUnknown;
    if (e->device != stub().device[std::this_thread::get_id()]) stub().event_mismatches++;
    e->pending = true;
    stub_op op;
    op.event = e;
    stub().queue[stub_runtime::key(s)].push_back(op);
    return hipSuccess;
}
inline hipError_t hipEventSynchronize(hipEvent_t e)
{
    std::lock_guard<std::mutex> l(stub().mu);
    for (auto &q : stub().queue)
        if (e->pending)
            for (const stub_op &op : q.second)
                if (op.event == e) {
                    stub_runtime::run(q.second, e);
                    break;
                }
    return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t s)
{
    std::lock_guard<std::mutex> l(stub().mu);
    stub_runtime::run(stub().queue[stub_runtime::key(s)], nullptr);
    return hipSuccess;
}
inline hipError_t stub_enqueue(void *dst, const void *src, size_t n, hipStream_t s)
{
    std::lock_guard<std::mutex> l(stub().mu);
    if (src) stub().copied_by.push_back(std::this_thread::get_id());
    stub_op op;
    op.dst = dst;
    op.src = src;
    op.bytes = n;
    stub().queue[stub_runtime::key(s)].push_back(op);
    return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind, hipStream_t s)
{
    return stub_enqueue(dst, src, n, s);
}
inline hipError_t hipMemsetAsync(void *dst, int, size_t n, hipStream_t s) { return stub_enqueue(dst, nullptr, n, s); }
