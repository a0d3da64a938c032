// CPU tests of ppml_transfer.hpp over the stand-in runtime: one per argument.
#include "../../paper_1607_01105_amd/csrc/ppml_transfer.hpp"

#include <cfenv>
#include <cstdio>
#include <limits>
#include <string>

using namespace ppml;

static int failures = 0;
#define CHECK(c)                                                         \
    do {                                                                 \
        if (!(c)) {                                                      \
            failures++;                                                  \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #c);          \
        }                                                                \
    } while (0)

static const hipStream_t OWN = (hipStream_t)0x1000;

static std::vector<double> numbers(size_t n, double first)
{
    std::vector<double> v(n);
    for (size_t i = 0; i < n; i++) v[i] = first + 0.5 * (double)(i % 4096);
    return v;
}

// Three arrays, the second absent, to the "device" and back.
template <typename T> static void round_trip(hipStream_t s, long long n, int device = 0)
{
    const std::vector<double> a = numbers((size_t)n, 1.0), b = numbers((size_t)n, 7.0);
    const double *src[3] = {a.data(), nullptr, b.data()};
    std::vector<T> dev((size_t)(3 * n), T(-1));
    XferHold hold;
    CHECK(xfer_upload<T>(device, s, src, 3, n, dev.data(), hold) == hipSuccess);
    hipStreamSynchronize(s);  // as the set calls do
    CHECK(hold.release() == hipSuccess);
    bool same = true;
    for (long long i = 0; i < n; i++)
        same = same && dev[i] == (T)a[i] && dev[n + i] == T(0) && dev[2 * n + i] == (T)b[i];
    CHECK(same);
    std::vector<double> back((size_t)(3 * n), -1.0);
    CHECK(xfer_download<T>(device, s, dev.data(), 3 * n, back.data()) == hipSuccess);
    same = true;
    for (long long i = 0; i < 3 * n; i++) same = same && back[i] == (double)dev[i];
    CHECK(same);
}

static void sizes()
{
    for (long long n : {1ll, 65536ll, 65537ll, 262144ll, 700001ll}) {
        round_trip<float>(OWN, n);
        round_trip<double>(OWN, n);
    }
}

static void several_calls()
{
    std::vector<std::thread> ts;
    for (int t = 0; t < 4; t++)
        ts.emplace_back([t] {
            for (int i = 0; i < 3; i++) round_trip<float>((hipStream_t)(size_t)(0x1000 * (t + 1)), 300000 + t);
        });
    for (std::thread &t : ts) t.join();
}

// hipStreamPerThread is another stream in every thread: only the caller's is
// ordered with the caller's work.
static void per_thread_stream()
{
    round_trip<float>(hipStreamPerThread, 700001);
    round_trip<double>(hipStreamPerThread, 700001);
    // work that is still queued there comes before a read
    const long long n = 700001;
    std::vector<float> old((size_t)n, 1.0f), stepped((size_t)n, 2.0f);
    std::vector<double> back((size_t)n);
    hipMemcpyAsync(old.data(), stepped.data(), (size_t)n * sizeof(float), hipMemcpyHostToDevice, hipStreamPerThread);
    CHECK(xfer_download<float>(0, hipStreamPerThread, old.data(), n, back.data()) == hipSuccess);
    bool fresh = true;
    for (double v : back) fresh = fresh && v == 2.0;
    CHECK(fresh);
    bool own = true;
    for (std::thread::id id : stub().copied_by) own = own && id == std::this_thread::get_id();
    CHECK(own);
}

// A copy whose event cannot be recorded has ended before its buffer goes back
// to the pool, and the call reports the error.
static void record_fails()
{
    const long long n = 700001;
    const std::vector<double> a = numbers((size_t)n, 1.0);
    const double *src[1] = {a.data()};
    std::vector<float> dev((size_t)n);
    std::vector<double> back((size_t)n);
    for (int down = 0; down < 2; down++)
        for (int k = 0; k < 3; k++) {
            stub().fail_record = stub().records + k;
            {
                XferHold hold;
                CHECK((down ? xfer_download<float>(0, OWN, dev.data(), n, back.data())
                            : xfer_upload<float>(0, OWN, src, 1, n, dev.data(), hold)) != hipSuccess);
            }
            for (const auto &q : stub().queue) CHECK(q.second.empty());
            stub().fail_record = -1;
            round_trip<float>(OWN, n);
        }
}

// The caller's floating-point environment reaches neither the conversions, which
// round to nearest as the device does, nor is it changed by them.
static void environment()
{
    std::vector<double> a(700001, 1.0 / 3.0);
    const long long n = (long long)a.size();
    const float nearest = (float)a[0];
    const double *src[1] = {a.data()};
    std::vector<float> dev(a.size());
    for (int mode : {FE_UPWARD, FE_DOWNWARD, FE_TOWARDZERO, FE_TONEAREST}) {
        std::feclearexcept(FE_ALL_EXCEPT);
        std::fesetround(mode);
        XferHold hold;
        const hipError_t e = xfer_upload<float>(0, OWN, src, 1, n, dev.data(), hold);
        const int after = std::fegetround(), raised = std::fetestexcept(FE_INEXACT);
        std::fesetround(FE_TONEAREST);
        CHECK(e == hipSuccess && after == mode && !raised && hold.release() == hipSuccess);
        bool same = true;
        for (float v : dev) same = same && v == nearest;
        CHECK(same);
    }
    a[n / 2] = std::numeric_limits<double>::quiet_NaN();
    feenableexcept(FE_INEXACT | FE_INVALID);
    XferHold hold;
    CHECK(xfer_upload<float>(0, OWN, src, 1, n / 2, dev.data(), hold) == hipSuccess);
    const bool finite = xfer_check(a.data(), n, false), positive = xfer_check(a.data(), n, true);
    fedisableexcept(FE_ALL_EXCEPT);
    CHECK(!finite && !positive);
    a[n / 2] = std::numeric_limits<double>::denorm_min();
    CHECK(xfer_check(a.data(), n, true));
}

// The buffers kept for one device serve another: no pinned memory is allocated
// anew, and every event is recorded on its own device.
static void devices()
{
    hipError_t e = hipSuccess;
    std::vector<XferLane *> lanes;
    for (size_t i = 0; i < XFER_IDLE; i++) lanes.push_back(xfer_pool().take(0, e));
    for (XferLane *l : lanes) xfer_pool().give(l);
    const int allocs = stub().host_allocs;
    for (int i = 0; i < 3; i++)
        for (int device = 0; device < 4; device++) round_trip<float>((hipStream_t)(size_t)(0x1000 + device), 700001, device);
    CHECK(stub().host_allocs == allocs);
    CHECK(stub().event_mismatches == 0);
}

// An upload does not wait for its copies, and no other call gets its buffers
// while they are held.
static void held()
{
    const long long n = 4096;
    const std::vector<double> a = numbers((size_t)n, 1.0), b = numbers((size_t)n, 7.0);
    const double *sa[1] = {a.data()}, *sb[1] = {b.data()};
    std::vector<float> da((size_t)n), db((size_t)n);
    {
        XferHold ha, hb;
        CHECK(xfer_upload<float>(0, OWN, sa, 1, n, da.data(), ha) == hipSuccess);
        CHECK(!stub().queue[stub_runtime::key(OWN)].empty());
        CHECK(xfer_upload<float>(0, OWN, sb, 1, n, db.data(), hb) == hipSuccess);
    }
    CHECK(stub().queue[stub_runtime::key(OWN)].empty());
    bool same = true;
    for (long long i = 0; i < n; i++) same = same && da[i] == (float)a[i] && db[i] == (float)b[i];
    CHECK(same);
}

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "sizes") sizes();
    else if (what == "several_calls") several_calls();
    else if (what == "per_thread_stream") per_thread_stream();
    else if (what == "record_fails") record_fails();
    else if (what == "environment") environment();
    else if (what == "devices") devices();
    else if (what == "held") held();
    else return 2;
    std::printf("%s: %d failure(s)\n", what.c_str(), failures);
    return failures != 0;
}
