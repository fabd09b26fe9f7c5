// A run of the modified-equilibrium model over an even number of steps ends in
// the caller's buffer by itself: no copy of the populations, whatever the steps
// per launch and per noise batch.  The runtime's calls are answered here, so
// nothing is launched and no GPU is needed.  Prints the number of runs with a
// copy too many and the first of them.

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>

#include "../include/flb.h"

static long copies = 0;

extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
extern "C" hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) {
    return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds,
                                                hipStream_t* st) {
    *grid = *block = dim3(1);
    *lds = 0;
    *st = nullptr;
    return hipSuccess;
}
extern "C" hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) {
    return hipSuccess;
}
extern "C" hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) {
    ++copies;
    return hipSuccess;
}

int main() {
    long runs = 0, bad = 0;
    // three, two and one step per launch
    const int box[][2] = {{64, 64}, {300, 300}, {1024, 1024}, {1024, 65}};
    for (const auto& n : box)
        for (int prec = 0; prec < 2; ++prec)
            for (double kT : {0.0, 1e-7})
                for (int batch : {1, 2, 3, 7, 16})
                    for (int steps = 0; steps <= 40; ++steps) {
                        flb_modeq_params p;
                        std::memset(&p, 0, sizeof p);
                        p.nx = n[0];
                        p.ny = n[1];
                        p.precision = prec;
                        p.rho0 = 1.0;
                        p.kT = kT;
                        p.cs2_0 = 0.07;
                        p.kappa = 0.08;
                        p.rate_bulk = p.rate_shear = p.rate_ghost = 1.0;
                        size_t w = 0;
                        if (flb_modeq_work_bytes(&p, &w) != FLB_OK) return 2;
                        copies = 0;
                        if (flb_modeq_run(&p, (void*)4096, (void*)8192, 0, steps, (void*)12288,
                                          w * batch, nullptr) != FLB_OK) {
                            std::printf("%s\n", flb_last_error());
                            return 2;
                        }
                        ++runs;
                        const long allowed = steps & 1;
                        if (copies > allowed && bad++ == 0)
                            std::printf("first: %d x %d prec %d kT %g batch %d: %d steps, a copy\n",
                                        n[0], n[1], prec, kT, batch, steps);
                    }
    std::printf("%ld runs, %ld with a copy too many\n", runs, bad);
    return bad != 0;
}
