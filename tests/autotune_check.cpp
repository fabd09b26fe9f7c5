// The autotuner's choices with every launch at a known cost: 3.6 us a step in
// launches of several D2Q9 steps, 3 us in in-place pairs of row tiles, 3.8 in all
// others, and 20 us once per timed trial.  A choice from a handful of launches
// sees mostly that once.  The runtime's calls are answered here, so nothing is
// launched and no GPU is needed.  Prints the launches of several steps in 24
// steps after it, the trials of several steps that drew the noise of a step drawn
// before, and the pairs chosen on a small thin box.

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>
#include <map>
#include <set>
#include <string>

#include "../include/flb.h"

static std::map<const void*, std::string>& kernels() {
    static std::map<const void*, std::string> m;
    return m;
}
static double now_us = 0.0;
static long several = 0, drawn_before = 0;
static std::set<unsigned long long> drawn;
static bool thin = false;
static const int T = 4;   // steps per launch of this box
static std::map<hipEvent_t, double> stamp;

extern "C" {
void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, uint3*,
                           uint3*, dim3*, dim3*, int*) {
    kernels()[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* st) {
    *grid = *block = dim3(1);
    *lds = 0;
    *st = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t) {
    const bool multi = kernels()[f].find("k_multi") != std::string::npos;
    several += multi;
    if (multi) {   // the fifth argument: the device counter (null here) and the host's index
        struct StepIndex {
            const unsigned long long* dev;
            unsigned long long host;
        } at;
        std::memcpy(&at, args[4], sizeof at);
        drawn_before += !drawn.insert(at.host).second;
    }
    const bool row_pair = thin && kernels()[f].find("k_step_ip") != std::string::npos;
    now_us += multi ? 3.6 * T : row_pair ? 3.0 : 3.8;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) {
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
    static char events[64];
    static int n = 0;
    *e = (hipEvent_t)&events[n++];
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
    stamp[e] = now_us;
    now_us += 10.0;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
    *ms = (float)((stamp[b] + 10.0 - stamp[a]) * 1e-3);
    return hipSuccess;
}
}

int main() {
    flb_params p;
    std::memset(&p, 0, sizeof p);
    p.lattice = FLB_D2Q9;
    p.precision = FLB_FP32;
    p.nx = p.ny = 256;
    p.nz = 1;
    p.force_model = FLB_IDEAL;
    p.rho0 = 1.0;
    p.kT = 1e-5;
    p.rate_bulk = 1.2;
    p.rate_shear = 1.6;
    p.rate_ghost = 1.0;
    for (int stats = 0; stats < 2; ++stats) {
        flb_handle* h = nullptr;
        if (flb_init(&p, (void*)4096, (void*)(1 << 24), (void*)(2 << 24), (void*)(3 << 24), nullptr,
                     nullptr, &h) != FLB_OK ||
            flb_autotune(h, 5, nullptr, nullptr, nullptr) != FLB_OK) {
            std::printf("%s\n", flb_last_error());
            return 2;
        }
        several = 0;
        const long trials_before = drawn_before;
        drawn.clear();
        if (flb_step(h, 24, stats, nullptr) != FLB_OK) return 2;
        std::printf("stride %d: %ld launches of several steps\n", stats, several);
        flb_destroy(h);
        drawn.clear();
        drawn_before = trials_before;
        if (several != 24 / T) return 1;
    }
    std::printf("%ld trials under noise drawn before\n", drawn_before);
    // a small box whose row tiles are three quarters empty: they are timed too
    thin = true;
    p.lattice = FLB_D3Q19;
    p.precision = FLB_FP64;
    p.nx = p.nz = 64;
    p.ny = 1;
    flb_handle* h = nullptr;
    int32_t best[4], shape[8];
    if (flb_init(&p, (void*)4096, (void*)(1 << 24), (void*)(2 << 24), (void*)(3 << 24), nullptr, nullptr,
                 &h) != FLB_OK ||
        flb_autotune(h, 5, best, nullptr, nullptr) != FLB_OK || best[3] < 0 ||
        flb_launch_shape(h, best[3], shape) != FLB_OK)
        return 2;
    std::printf("pairs of %s\n", shape[7] == 3 ? "consecutive sites" : "row tiles");
    flb_destroy(h);
    return 0;
}
