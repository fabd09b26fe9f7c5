// Every launch of the modified-equilibrium noise asks for no more dynamic LDS
// than the kernel's limit: 64 KB, or what hipFuncSetAttribute raised it to
// before.  The runtime's launch calls are answered here, so nothing is launched and
// no GPU is needed.  Prints the number of launches over their limit and the
// first of them.

#include <cstdio>
#include <map>

#include "../paper_1012_3632_amd/csrc/internal.h"

static std::map<const void*, size_t> limit;
static long launches = 0, bad = 0;
static int nx = 0, ny = 0, prec = 0;

extern "C" hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute attr, int value) {
    if (attr == hipFuncAttributeMaxDynamicSharedMemorySize) limit[f] = (size_t)value;
    return hipSuccess;
}

static dim3 cfg_grid, cfg_block;
static size_t cfg_lds = 0;

extern "C" hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t) {
    cfg_grid = grid;
    cfg_block = block;
    cfg_lds = lds;
    return hipSuccess;
}

extern "C" hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds,
                                                hipStream_t* st) {
    *grid = cfg_grid;
    *block = cfg_block;
    *lds = cfg_lds;
    *st = nullptr;
    return hipSuccess;
}

extern "C" hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t lds,
                                      hipStream_t) {
    const auto it = limit.find(f);
    const size_t most = it == limit.end() ? 65536 : it->second;
    ++launches;
    if ((lds > most || lds > flb::LDS_BYTES || grid.x == 0 || block.x == 0 || block.x > 1024) &&
        bad++ == 0)
        std::printf("first: %d x %d prec %d: %zu bytes, limit %zu, %u threads\n", nx, ny, prec, lds,
                    most, block.x);
    return hipSuccess;
}

int main() {
    auto look = [&](int x, int y) {
        flb::ModEqArgs a{};
        a.nx = nx = x;
        a.ny = ny = y;
        a.prec = prec;
        for (int nb : {1, flb::MODEQ_MAX_BATCH}) {
            limit.clear();   // the limits a call relies on are the ones it raises
            (void)flb::launch_modeq_noise(a, prec, 0, nb, nullptr, nullptr, nullptr);
        }
    };
    for (prec = 0; prec < 2; ++prec)
        for (int n = 1; n <= 1024; ++n)
            for (int m : {1, 126, 1024}) {
                look(n, m);
                look(m, n);
            }
    std::printf("%ld launches, %ld over their limit\n", launches, bad);
    return bad != 0 || launches == 0;
}
