// Which kernels vp_project launches, without a GPU: as in kmeans_launch_main.cpp the HIP calls that the library makes are
// defined here, in front of the runtime's, and launched kernels are written down instead of run.
// usage: project_launch <d> <V> <K> <lo> <hi> <k> <N>...: an index of K active sets of lo to hi tokens, evenly spaced; for
// every N prints a line "N status" and then one line per kernel: its name and its workgroups.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
#include <utility>
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
std::vector<std::pair<std::string, uint32_t>> launched;
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
int hipLaunchKernel(const void *f, Dim3 grid, Dim3, void **, size_t, void *)
{
    launched.emplace_back(names()[f], grid.x * grid.y);
    return 0;
}
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetLastError(void) { return 0; }
int hipMemcpyAsync(void *, const void *, size_t, int, void *) { return 0; }
int hipMemsetAsync(void *, int, size_t, void *) { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipGetSymbolAddress(void **p, const void *)
{
    *p = reinterpret_cast<void *>(4096);
    return 0;
}
int hipGetDevice(int *dev)
{
    *dev = 0;
    return 0;
}
int hipDeviceGetAttribute(int *value, int, int)
{
    *value = 256;   // (only the compute units are asked for)
    return 0;
}

}  // extern "C"

int main(int argc, char **argv)
{
    if (argc < 8) return 2;
    const int K = std::atoi(argv[3]), lo = std::atoi(argv[4]), hi = std::atoi(argv[5]), k = std::atoi(argv[6]);
    std::vector<int64_t> offsets(1, 0);
    std::vector<int32_t> ids;
    for (int j = 0; j < K; ++j) {
        const int n = lo + (int)((int64_t)(hi - lo) * j / (K > 1 ? K - 1 : 1));
        for (int i = 0; i < n; ++i) ids.push_back(i);
        offsets.push_back((int64_t)ids.size());
    }
    void *const some = reinterpret_cast<void *>(4096);   // (aligned; nobody follows it)
    vp_build_desc D = {};
    D.d = std::atoi(argv[1]);
    D.V = std::atoi(argv[2]);
    D.K = K;
    D.W = D.bias = D.centroids = D.arena = some;
    D.cand_offsets = offsets.data();
    D.cand_ids = ids.data();
    D.k_max = 8;
    D.arena_bytes = vp_build_bytes(&D);
    vp_index *index = nullptr;
    if (vp_build(&D, nullptr, &index) != VP_OK) {
        std::fprintf(stderr, "%s\n", vp_last_error());
        return 3;
    }
    for (int a = 7; a < argc; ++a) {
        const int N = std::atoi(argv[a]);
        launched.clear();
        const vp_status s = vp_project(index, some, N, k, (int32_t *)some, (float *)some, nullptr, some,
                                       vp_workspace_bytes(index, N), nullptr);
        std::printf("%d %d\n", N, (int)s);
        for (const auto &l : launched) std::printf("%s %u\n", l.first.c_str(), l.second);
    }
    return 0;
}
