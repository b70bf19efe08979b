// Which kernels vp_kmeans launches, without a GPU: this program defines the HIP calls that the library
// launches through, in front of the runtime's, and writes every launched kernel's name down instead of
// running it.  usage: kmeans_launch <fail_attribute> <n> <d> <K> <iters>; prints the status, the number of
// hipFuncSetAttribute calls, the error left behind, then one kernel name a line.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
#include <vector>

#include "vp.h"

namespace {

struct Dim3 {
    uint32_t x, y, z;
};

std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m;   // (filled by the library's constructors, before main)
    return m;
}
std::vector<std::string> launched;
bool fail_attribute = false;
int attribute_calls = 0;
int last_error = 0;
struct {
    Dim3 grid, block;
    size_t shared;
    void *stream;
} pushed;

}  // namespace

extern "C" {

void __hipRegisterFunction(void *, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *)
{
    names()[host] = name;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void *stream)
{
    pushed = {grid, block, shared, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *shared, void **stream)
{
    *grid = pushed.grid;
    *block = pushed.block;
    *shared = pushed.shared;
    *stream = pushed.stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim3, Dim3, void **, size_t, void *)
{
    launched.push_back(names()[f]);
    return 0;
}
int hipFuncSetAttribute(const void *, int, int)
{
    ++attribute_calls;
    if (!fail_attribute) return 0;
    last_error = 1;
    return 1;
}
int hipGetLastError(void)
{
    const int e = last_error;
    last_error = 0;
    return e;
}

}  // extern "C"

int main(int argc, char **argv)
{
    if (argc != 6) return 2;
    fail_attribute = std::atoi(argv[1]) != 0;
    const int64_t n = std::atoll(argv[2]);
    const int d = std::atoi(argv[3]), K = std::atoi(argv[4]), iters = std::atoi(argv[5]);
    void *const some = reinterpret_cast<void *>(4096);   // (aligned; nobody follows it)
    const vp_status s = vp_kmeans(some, n, d, K, iters, 0, some, (int32_t *)some, (int32_t *)some, some,
                                  vp_kmeans_workspace_bytes(n, d, K), nullptr);
    std::printf("%d\n%d\n%d\n", (int)s, attribute_calls, last_error);
    for (const std::string &name : launched) std::printf("%s\n", name.c_str());
    return 0;
}
