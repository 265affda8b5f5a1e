// miconv_stack_create where device memory is short, without a GPU: this program
// stands in for the HIP runtime calls that create makes (its own definitions
// take precedence over the library's) and lets hipMalloc fail above a size.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>

#include "miconv.h"

namespace {
size_t limit = ~(size_t)0;
std::set<void *> live;
int last_error = 0, objects = 0;
int fail(int e) { return last_error = e; }
}  // namespace

struct Dim3 {
    unsigned x, y, z;
};

extern "C" {
int hipGetDevice(int *d) { return *d = 0; }
int hipDeviceGetAttribute(int *v, int, int) { return *v = 256, 0; }
int hipMalloc(void **p, size_t n)
{
    if (n > limit) return fail(2);                        // hipErrorOutOfMemory
    *p = std::aligned_alloc(256, 256);                    // never dereferenced
    live.insert(*p);
    return 0;
}
int hipFree(void *p)
{
    if (!live.erase(p)) std::abort();
    std::free(p);
    return 0;
}
int hipGetLastError()
{
    const int e = last_error;
    last_error = 0;
    return e;
}
int hipStreamSynchronize(void *) { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { return ++objects, *s = &objects, 0; }
int hipStreamDestroy(void *) { return --objects, 0; }
int hipEventCreateWithFlags(void **e, unsigned) { return ++objects, *e = &objects, 0; }
int hipEventDestroy(void *) { return --objects, 0; }
int __hipPushCallConfiguration(Dim3, Dim3, size_t, void *) { return 0; }
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *m, void **s)
{
    *g = *b = Dim3{1, 1, 1};
    return *m = 0, *s = nullptr, 0;
}
int hipLaunchKernel(const void *, Dim3, Dim3, void **, size_t, void *) { return 0; }
}

int main()
{
    // two layers that do not depend on each other; the first runs on a split copy of x
    auto at = [](size_t mb) { return reinterpret_cast<void *>(mb << 20); };
    miconv_conv_desc d[2] = {};
    d[0] = {MICONV_OP_CONV_F32, 16, 128, 56, 56, 256, 3, 3, 1, 1, 1, 1, at(100), at(300), nullptr, at(400), nullptr, 0, 0};
    d[1] = {MICONV_OP_CONV_F32, 1, 512, 7, 7, 512, 3, 3, 1, 1, 1, 1, at(600), at(700), nullptr, at(800), nullptr, 0, 0};
    const struct {
        size_t limit;
        int rc;
        const char *kernel;
    } cases[] = {{~(size_t)0, MICONV_OK, "igemm_split3"}, {20u << 20, MICONV_OK, "igemm_wave"}, {0, MICONV_ERR_HIP, ""}};
    for (const auto &c : cases) {
        limit = c.limit;
        miconv_stack *s = nullptr;
        const int rc = miconv_stack_create(d, 2, &s);
        char name[512] = "";
        if (s) miconv_stack_describe(s, 0, name, sizeof name);
        if (rc != c.rc || (s != nullptr) != (rc == MICONV_OK) || !std::strstr(name, c.kernel)) {
            std::printf("limit %zu: rc %d %s\n", c.limit, rc, name);
            return 1;
        }
        miconv_stack_destroy(s);
        if (!live.empty() || objects) {
            std::printf("limit %zu: %zu allocations, %d objects left\n", c.limit, live.size(), objects);
            return 1;
        }
        hipGetLastError();
    }
    std::printf("ok\n");
    return 0;
}
