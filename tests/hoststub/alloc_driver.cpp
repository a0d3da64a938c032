// Heap allocations of the grid set-up that the allocation-free entry point goes
// through: includes the implementation, whose set-up functions are internal.
#include "../../paper_1607_01105_amd/csrc/ppml_api.hip"

#include <cstdio>
#include <cstdlib>

// (linked without the HIP runtime: nothing here calls it)
extern "C" {
void **__hipRegisterFatBinary(const void *) { return nullptr; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
}

static long long allocations = 0;

void *operator new(size_t n)
{
    allocations++;
    void *p = std::malloc(n);
    if (!p) std::abort();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

int main()
{
    int failures = 0;
    for (int ndim = 1; ndim <= 3; ndim++)
        for (int prec : {PPML_FP32, PPML_FP64})
            for (int n : {3, 40, 300}) {
                GridParams gp{};
                gp.ndim = ndim;
                for (int a = 0; a < 3; a++) gp.n[a] = a < ndim ? n : 1;
                const long long before = allocations;
                set_tiling(gp, ndim, prec, 0);
                if (allocations != before) {
                    failures++;
                    std::printf("%d-D precision %d, %d cells an axis: %lld allocations\n", ndim, prec, n, allocations - before);
                }
            }
    std::printf("%d failure(s)\n", failures);
    return failures != 0;
}
