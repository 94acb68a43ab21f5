// Rules of the several-gates-per-sweep path (tile.h) that hold without a GPU.
//
//   tile_rules layout     the programs lie at multiples of 16 bytes
#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../paper_2511_19291_amd/csrc/tile.h"

namespace sv {
void launch_tile_adj(const TileAdjArgs&, int, int, hipStream_t) {}
void launch_sum_slots(const double*, int, int, double*, hipStream_t) {}
void launch_tile(const TileArgs&, int, int, hipStream_t) {}
void fail(sv_status, const std::string& msg)
{
    std::fprintf(stderr, "%s\n", msg.c_str());
    std::abort();
}
void hip_check(hipError_t, const char*) {}
const DeviceInfo& device_info()
{
    static DeviceInfo d;
    d.cu_count = 256;
    return d;
}
}  // namespace sv

// The kernels read headers and matrices as 16-byte words from `words` on; the
// kernel arguments themselves lie at a multiple of 16.
static int layout()
{
    const size_t run = offsetof(sv::TileArgs, words), adj = offsetof(sv::TileAdjArgs, words);
    std::printf("words at %zu and %zu\n", run, adj);
    return run % 16 == 0 && adj % 16 == 0 && alignof(sv::TileArgs) % 16 == 0 && alignof(sv::TileAdjArgs) % 16 == 0 ? 0 : 1;
}

int main(int argc, char** argv)
{
    if (argc != 2) return 2;
    if (!std::strcmp(argv[1], "layout")) return layout();
    return 2;
}
