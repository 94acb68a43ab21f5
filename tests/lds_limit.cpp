// The limit of dynamic LDS that a kernel is given is a property of the function,
// shared by every thread and stream: each call has to set the same one, and no
// launch may need more. Linked with the library's kernels, HIP's calls replaced.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <memory>
#include <set>
#include <string>

#include "../paper_2511_19291_amd/csrc/batch.h"
#include "../paper_2511_19291_amd/csrc/tile.h"

static std::map<const void*, std::set<int>> limits;    // every limit that a function was given
static std::map<const void*, size_t> most;             // the most that a launch took

extern "C" hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int value)
{
    limits[f].insert(value);
    return hipSuccess;
}
// (what <<<>>> keeps between a launch's configuration and its stub)
static size_t configured;
extern "C" hipError_t __hipPushCallConfiguration(dim3, dim3, size_t lds, hipStream_t)
{
    configured = lds;
    return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* st)
{
    *grid = *block = dim3(1);
    *lds = configured;
    *st = nullptr;
    return hipSuccess;
}
extern "C" hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t lds, hipStream_t)
{
    most[f] = std::max(most[f], lds);
    return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
extern "C" hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int, size_t lds)
{
    most[f] = std::max(most[f], lds);
    *n = 1;
    return hipSuccess;
}

namespace sv {
void fail(sv_status, const std::string& msg)
{
    std::fprintf(stderr, "%s\n", msg.c_str());
    std::abort();
}
void hip_check(hipError_t, const char*) {}
}  // namespace sv

int main()
{
    auto a = std::make_unique<sv::TileAdjArgs>();
    // a state in one tile and one of many, with many values and with few
    for (int n : {12, 20})
        for (int values : {n == 12 ? sv::kAdjValues : sv::kAdjTileValues, 1, 60, 0}) {
            a->N = 1ull << n;
            a->T = 12;
            a->nvalues = values;
            sv::launch_tile_adj(*a, 1, 1, nullptr);
        }
    // plans of narrow tiles made after plans of wide ones
    for (int bits = sv::kMaxTileBits; bits >= sv::kMinTileBits; --bits)
        for (int threads : {256, 512, 1024})
            for (int mode = 0; mode < 3; ++mode) sv::batch_max_wg_per_cu(threads, bits, mode);
    std::printf("%zu kernels launched, %zu given a limit\n", most.size(), limits.size());
    if (most.size() != 2 + 9 || limits.size() != most.size()) return 1;
    for (const auto& m : most) {
        const std::set<int>& l = limits[m.first];
        std::printf("%zu limits, %d bytes, at most %zu taken\n", l.size(), *l.begin(), m.second);
        if (l.size() != 1 || (size_t)*l.begin() < m.second || *l.begin() > 160 * 1024) return 1;
    }
    return 0;
}
