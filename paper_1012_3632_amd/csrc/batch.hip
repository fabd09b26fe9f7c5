// Batched replicas: many independent ideal-gas lattices of uneven size
// advanced by one launch per step.
//
// Every replica's sites are cut into tiles of BT = 256 consecutive sites
// (x fastest; the last tile of a replica may be partly empty), the tiles of
// all replicas form one flat table, and a block takes one tile, the flat step
// of flat.h.  Replica r has its own box, Philox key seeds[r] and counter word
// 3 = r, and its populations start at element Q * sum_{s<r} V_s of each buffer.
// In-place pairs (optional, flb_batch_set_pairs): consecutive replicas are
// grouped up to a byte budget and each group is taken through all the steps of
// a call before the next, pairs of steps in one buffer (the first step of a
// pair stores S*_i(x) in plane opp(i) at x + c_i, the second reads plane
// opp(i) at x and stores plane i at x; every location a thread writes is one
// only it reads, just before), so that a group's working set can stay in the
// last-level cache.  The noise counters hold the global step, so the result
// is the same bits in either schedule.
// Statistics: a sampled step adds each tile's 2Q FP64 block sums to the tile's
// own slots, and at the end of a call k_batch_fold adds, per replica and value,
// the sum over the replica's tiles (fixed order) to an FP64 accumulator and
// clears the slots.  Either schedule adds the same tile sums in the same step
// order, so the statistics are bitwise the same.
//
// A block per tile rather than a persistent grid over chunks of eight tiles
// with sums kept across them: a group near the cache size has about 1200
// chunks, barely more than fit the chip at once, so its last wave of blocks
// left it nearly idle, and the kept sums cost a third of the wavefronts.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/flb.h"
#include "device.h"
#include "flat.h"
#include "internal.h"

namespace flb {

constexpr int BT = FLAT_NT;   // sites per tile (one per thread)

struct RepInfo {
    int32_t nx, ny, nz;
    uint32_t V;
    uint64_t off;          // element offset of the replica in a population buffer
    uint32_t key0, key1;
    uint32_t tile0, ntiles;
    uint32_t inv_nx, inv_ny;   // ceil(2^32 / n): exact division for n < 256, s < 2^24
};

// The tiles from t0 on: KIND 0 from fin to fout, 1 and 2 the phases of an
// in-place pair (fin == fout, not restrict: a thread's stores alias its own
// earlier loads).
template <int LAT, typename Real, bool STATS, int KIND>
__global__ __launch_bounds__(BT) void k_batch_step(const Real* fin, Real* fout,
                                                   const RepInfo* __restrict__ reps,
                                                   const uint32_t* __restrict__ tile_rep,
                                                   uint32_t t0, CollideParams<Real> P, StepIndex st,
                                                   double* __restrict__ partial) {
    constexpr int Q = Lattice<LAT>::Q;
    __shared__ double lds_stats[STATS ? 4 * (BT / 64) * 2 * Q : 1];
    const double2* tab = noise_table<Real, BT>();
    const uint32_t t = t0 + xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t r = tile_rep[t];
    const RepInfo R = reps[r];
    const uint32_t s = (t - R.tile0) * (uint32_t)BT + threadIdx.x;
    const uint32_t step = st.get();
    Real v[STATS ? 2 * Q : 1];
    if constexpr (STATS) {
#pragma unroll
        for (int k = 0; k < 2 * Q; ++k) v[k] = Real(0);
    }
    if (s < R.V)
        flat_site<LAT, Real, STATS, KIND>(fin + R.off, fout + R.off, s,
                                          FlatBox{R.nx, R.ny, R.nz, R.V, R.inv_nx, R.inv_ny}, P, r,
                                          R.key0, R.key1, step, tab, v);
    if constexpr (STATS) block_accumulate<2 * Q, BT>(v, partial + (size_t)t * 2 * Q, lds_stats);
}

// acc[r][k] += sum over replica r's tiles (fixed order) of partial[tile][k],
// then those slots are cleared.  One block per (value k, replica r).
__global__ void k_batch_fold(double* __restrict__ partial, const RepInfo* __restrict__ reps,
                             int nvals, double* __restrict__ acc_out) {
    __shared__ double red[256];
    const int k = blockIdx.x, r = blockIdx.y;
    const RepInfo R = reps[r];
    double* col = partial + (size_t)R.tile0 * nvals + k;
    double acc = 0.0;
    for (uint32_t t = threadIdx.x; t < R.ntiles; t += 256) {
        acc += col[(size_t)t * nvals];
        col[(size_t)t * nvals] = 0.0;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) acc_out[(size_t)r * nvals + k] += red[0];
}

}  // namespace flb

using namespace flb;

namespace {

flb_status bfail(flb_status s, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    set_last_error(buf);
    return s;
}

#define BHIP(expr)                                                                        \
    do {                                                                                  \
        hipError_t e_ = (expr);                                                           \
        if (e_ != hipSuccess)                                                             \
            return bfail(FLB_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(e_));     \
    } while (0)

constexpr size_t ALIGN = 256;
size_t align_up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }
constexpr double CS2 = 1.0 / 3.0;

struct Layout {
    std::vector<RepInfo> reps;
    std::vector<uint32_t> tile_rep;
    size_t elems;          // reals per population buffer
    size_t reps_off, tiles_off, ctr_off, scratch_bytes, stats_bytes;
};

flb_status batch_layout(const flb_params* p, int32_t nrep, const int32_t* dims,
                        const uint64_t* seeds, Layout* L) {
    if (!p || !dims) return bfail(FLB_ERR_INVALID_ARG, "NULL argument");
    if (nrep < 1 || nrep > 4096) return bfail(FLB_ERR_INVALID_ARG, "nrep = %d", nrep);
    if (p->force_model != FLB_IDEAL)
        return bfail(FLB_ERR_UNSUPPORTED, "batched replicas are ideal-gas only");
    flb_params q = *p;
    const int Q = p->lattice == FLB_D2Q9 ? 9 : 19;
    L->reps.clear();
    L->tile_rep.clear();
    size_t off = 0;
    uint32_t tile = 0;
    for (int r = 0; r < nrep; ++r) {
        q.nx = dims[3 * r];
        q.ny = dims[3 * r + 1];
        q.nz = dims[3 * r + 2];
        size_t a, b, c;
        flb_status st = flb_query_sizes(&q, &a, &b, &c);
        if (st != FLB_OK) {
            const std::string why = flb_last_error();
            return bfail(st, "replica %d: %s", r, why.c_str());
        }
        if (q.nx >= 256 || q.ny >= 256 || q.nz >= 65536)
            return bfail(FLB_ERR_INVALID_ARG, "replica %d: batched boxes need nx, ny < 256", r);
        RepInfo R{};
        R.nx = q.nx;
        R.ny = q.ny;
        R.nz = q.nz;
        R.V = (uint32_t)q.nx * q.ny * q.nz;
        if (R.V >= (1u << 24)) return bfail(FLB_ERR_INVALID_ARG, "replica %d too large", r);
        R.off = off;
        const uint64_t seed = seeds ? seeds[r] : (uint64_t)r;
        R.key0 = (uint32_t)(seed & 0xffffffffu);
        R.key1 = (uint32_t)(seed >> 32);
        R.tile0 = tile;
        R.ntiles = (R.V + BT - 1) / BT;
        R.inv_nx = (uint32_t)(((1ull << 32) + R.nx - 1) / R.nx);
        R.inv_ny = (uint32_t)(((1ull << 32) + R.ny - 1) / R.ny);
        L->tile_rep.insert(L->tile_rep.end(), R.ntiles, (uint32_t)r);
        tile += R.ntiles;
        off += (size_t)Q * R.V;
        L->reps.push_back(R);
    }
    L->elems = off;
    size_t s = 0;
    L->ctr_off = s;
    s += ALIGN;
    L->reps_off = s;
    s += align_up(L->reps.size() * sizeof(RepInfo));
    L->tiles_off = s;
    s += align_up(L->tile_rep.size() * sizeof(uint32_t));
    L->scratch_bytes = s;
    L->stats_bytes = align_up(((size_t)tile * 2 * Q + (size_t)nrep * 2 * Q) * sizeof(double));
    return FLB_OK;
}

}  // namespace

// The tiles [t0, t1) of consecutive replicas.
struct BatchGroup {
    uint32_t t0, t1;
};

struct flb_batch {
    flb_params p;
    int q, nrep;
    size_t rb;
    Layout L;
    void* fa;
    void* fb;
    bool cur_a;
    char* scratch;
    double* stats;
    RepInfo* reps_dev;
    uint32_t* tiles_dev;
    unsigned long long* ctr_dev;
    uint32_t ntiles;
    uint64_t step;
    int64_t nsamples;
    uint64_t pair_bytes;   // > 0: in-place pairs, groups of replicas up to this many bytes
    std::vector<BatchGroup> groups;
    // captured steps, one graph per current buffer (index cur_a): kernel
    // arguments hold the buffer pointers
    hipGraph_t graph[2];
    hipGraphExec_t gexec[2];
    int64_t graph_steps, graph_samples;
    void* cur() const { return cur_a ? fa : fb; }
    void* other() const { return cur_a ? fb : fa; }
};

namespace {

void release_batch_graphs(flb_batch* b) {
    for (int k = 0; k < 2; ++k) {
        if (b->gexec[k]) (void)hipGraphExecDestroy(b->gexec[k]);
        if (b->graph[k]) (void)hipGraphDestroy(b->graph[k]);
        b->gexec[k] = nullptr;
        b->graph[k] = nullptr;
    }
}

template <int LAT, typename Real>
CollideParams<Real> batch_collide_params(const flb_batch* b) {
    CollideParams<Real> P;
    const flb_params& p = b->p;
    P.rho0 = (Real)p.rho0;
    P.lam_bulk = (Real)p.rate_bulk;
    P.lam_shear = (Real)p.rate_shear;
    P.lam_ghost = (Real)p.rate_ghost;
    const double lam[3] = {p.rate_bulk, p.rate_shear, p.rate_ghost};
    for (int c = 0; c < 3; ++c)
        P.amp_cls[c] = (Real)std::sqrt(p.kT * lam[c] * (2.0 - lam[c]) / CS2);
    P.noise_on = p.kT > 0.0;
    P.noise_local = p.noise_rho_local ? 1 : 0;
    P.key0 = P.key1 = 0;   // per replica
    P.replica = 0;
    P.nonfinite = nullptr;
    return P;
}

// kind 0: all replicas from fin to fout; 1, 2: a phase of an in-place pair on
// the tiles of G (fin == fout).
template <int LAT, typename Real>
void batch_launch(flb_batch* b, int kind, const BatchGroup& G, const void* fin, void* fout,
                  const unsigned long long* step_dev, unsigned long long step_host,
                  double* partial, hipStream_t st) {
    const CollideParams<Real> P = batch_collide_params<LAT, Real>(b);
    StepIndex si{step_dev, step_host};
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(G.t1 - G.t0), dim3(BT), 0, st, (const Real*)fin, (Real*)fout,
                           b->reps_dev, b->tiles_dev, G.t0, P, si, partial);
    };
    if (kind == 0) partial ? go(k_batch_step<LAT, Real, true, 0>) : go(k_batch_step<LAT, Real, false, 0>);
    else if (kind == 1) partial ? go(k_batch_step<LAT, Real, true, 1>) : go(k_batch_step<LAT, Real, false, 1>);
    else partial ? go(k_batch_step<LAT, Real, true, 2>) : go(k_batch_step<LAT, Real, false, 2>);
}

hipError_t batch_one(flb_batch* b, int kind, const BatchGroup& G, const void* fin, void* fout,
                     const unsigned long long* step_dev, unsigned long long step_host,
                     double* partial, hipStream_t st) {
    const int lat = b->p.lattice, prec = b->p.precision;
    if (lat == 0 && prec == 0) batch_launch<0, float>(b, kind, G, fin, fout, step_dev, step_host, partial, st);
    else if (lat == 0) batch_launch<0, double>(b, kind, G, fin, fout, step_dev, step_host, partial, st);
    else if (prec == 0) batch_launch<1, float>(b, kind, G, fin, fout, step_dev, step_host, partial, st);
    else batch_launch<1, double>(b, kind, G, fin, fout, step_dev, step_host, partial, st);
    return hipGetLastError();
}

BatchGroup batch_all(const flb_batch* b) { return BatchGroup{0, b->ntiles}; }

// Consecutive replicas up to `bytes` of populations per group (a replica
// larger than that forms a group of its own).
std::vector<BatchGroup> batch_groups(const flb_batch* b, uint64_t bytes) {
    std::vector<BatchGroup> out;
    const std::vector<RepInfo>& R = b->L.reps;
    uint32_t r0 = 0;
    uint64_t acc = 0;
    for (uint32_t r = 0; r < (uint32_t)R.size(); ++r) {
        const uint64_t rb = (uint64_t)b->q * R[r].V * b->rb;
        if (r > r0 && acc + rb > bytes) {
            out.push_back({R[r0].tile0, R[r].tile0});
            r0 = r;
            acc = 0;
        }
        acc += rb;
    }
    out.push_back({R[r0].tile0, b->ntiles});
    return out;
}

double* batch_acc(flb_batch* b) { return b->stats + (size_t)b->ntiles * 2 * b->q; }

flb_status batch_run(flb_batch* b, int64_t nsteps, int32_t stride, bool graph_mode,
                     hipStream_t st, int64_t* samples) {
    int64_t ns = 0;
    const int nv = 2 * b->q;
    auto sampled = [stride](int64_t k) { return stride > 0 && ((k + 1) % stride) == 0; };
    auto index = [&](int64_t k) {
        return graph_mode ? (unsigned long long)k : (unsigned long long)(b->step + k);
    };
    const unsigned long long* sd = graph_mode ? b->ctr_dev : nullptr;
    int64_t k = 0;
    if (b->pair_bytes > 0 && nsteps >= 2) {
        // group by group, pairs of steps in place in the current buffer
        const int64_t np = nsteps & ~(int64_t)1;
        for (const BatchGroup& G : b->groups) {
            for (int64_t j = 0; j < np; ++j) {
                const bool sample = sampled(j);
                BHIP(batch_one(b, 1 + (int)(j & 1), G, b->cur(), b->cur(), sd, index(j),
                               sample ? b->stats : nullptr, st));
            }
        }
        for (int64_t j = 0; j < np; ++j) ns += sampled(j);
        k = np;
    }
    for (; k < nsteps; ++k) {
        const bool sample = sampled(k);
        BHIP(batch_one(b, 0, batch_all(b), b->cur(), b->other(), sd, index(k),
                       sample ? b->stats : nullptr, st));
        b->cur_a = !b->cur_a;
        ns += sample;
    }
    if (ns > 0) {
        hipLaunchKernelGGL(k_batch_fold, dim3(nv, b->nrep), dim3(256), 0, st, b->stats,
                           b->reps_dev, nv, batch_acc(b));
        BHIP(hipGetLastError());
    }
    if (graph_mode) BHIP(launch_add_u64(b->ctr_dev, (unsigned long long)nsteps, st));
    *samples = ns;
    return FLB_OK;
}

}  // namespace

extern "C" {

flb_status flb_batch_query_sizes(const flb_params* base, int32_t nrep, const int32_t* dims,
                                 size_t* pop_bytes, size_t* scratch_bytes, size_t* stats_bytes) {
    Layout L;
    flb_status s = batch_layout(base, nrep, dims, nullptr, &L);
    if (s != FLB_OK) return s;
    const size_t rb = base->precision == FLB_FP64 ? 8 : 4;
    if (pop_bytes) *pop_bytes = align_up(L.elems * rb);
    if (scratch_bytes) *scratch_bytes = L.scratch_bytes;
    if (stats_bytes) *stats_bytes = L.stats_bytes;
    return FLB_OK;
}

flb_status flb_batch_init(const flb_params* base, int32_t nrep, const int32_t* dims,
                          const uint64_t* seeds, void* f_a, void* f_b, void* scratch,
                          void* stats, void* stream, flb_batch** out) {
    if (!out) return bfail(FLB_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    auto al = [](const void* q) { return q && ((uintptr_t)q % ALIGN) == 0; };
    if (!al(f_a) || !al(f_b) || !al(scratch) || !al(stats) || f_a == f_b)
        return bfail(FLB_ERR_INVALID_ARG, "buffers must be distinct, non-NULL, 256-byte aligned");
    flb_batch* b = new (std::nothrow) flb_batch();
    if (!b) return bfail(FLB_ERR_INVALID_ARG, "out of host memory");
    flb_status s = batch_layout(base, nrep, dims, seeds, &b->L);
    if (s != FLB_OK) {
        delete b;
        return s;
    }
    hipStream_t st = (hipStream_t)stream;
    b->p = *base;
    b->q = base->lattice == FLB_D2Q9 ? 9 : 19;
    b->nrep = nrep;
    b->rb = base->precision == FLB_FP64 ? 8 : 4;
    b->fa = f_a;
    b->fb = f_b;
    b->cur_a = true;
    b->scratch = (char*)scratch;
    b->stats = (double*)stats;
    b->reps_dev = (RepInfo*)(b->scratch + b->L.reps_off);
    b->tiles_dev = (uint32_t*)(b->scratch + b->L.tiles_off);
    b->ctr_dev = (unsigned long long*)(b->scratch + b->L.ctr_off);
    b->ntiles = (uint32_t)b->L.tile_rep.size();
    b->step = base->step0;
    b->nsamples = 0;
    b->pair_bytes = 0;
    b->graph[0] = b->graph[1] = nullptr;
    b->gexec[0] = b->gexec[1] = nullptr;
    hipError_t e = hipSuccess;
    if (e == hipSuccess)
        e = hipMemcpyAsync(b->reps_dev, b->L.reps.data(), b->L.reps.size() * sizeof(RepInfo),
                           hipMemcpyHostToDevice, st);
    if (e == hipSuccess)
        e = hipMemcpyAsync(b->tiles_dev, b->L.tile_rep.data(), b->ntiles * sizeof(uint32_t),
                           hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = launch_set_u64(b->ctr_dev, b->step, st);
    if (e == hipSuccess) e = launch_fill_zero(stats, b->L.stats_bytes, st);
    // the uniform rest state: every deviation from w_i rho0 is zero
    if (e == hipSuccess) e = launch_fill_zero(f_a, b->L.elems * b->rb, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        delete b;
        return bfail(FLB_ERR_HIP, "flb_batch_init: %s", hipGetErrorString(e));
    }
    *out = b;
    return FLB_OK;
}

flb_status flb_batch_step(flb_batch* b, int64_t nsteps, int32_t stats_stride, void* stream) {
    if (!b) return bfail(FLB_ERR_INVALID_ARG, "batch is NULL");
    if (nsteps < 0 || stats_stride < 0) return bfail(FLB_ERR_INVALID_ARG, "bad step count");
    int64_t ns = 0;
    flb_status s = batch_run(b, nsteps, stats_stride, false, (hipStream_t)stream, &ns);
    if (s != FLB_OK) return s;
    b->step += (uint64_t)nsteps;
    b->nsamples += ns;
    BHIP(launch_set_u64(b->ctr_dev, b->step, (hipStream_t)stream));
    return FLB_OK;
}

flb_status flb_batch_moments(flb_batch* b, double* mode_sum, double* mode_sumsq,
                             int64_t* nsamples, void* stream) {
    if (!b) return bfail(FLB_ERR_INVALID_ARG, "batch is NULL");
    hipStream_t st = (hipStream_t)stream;
    const int nv = 2 * b->q;
    const double* out = batch_acc(b);
    std::vector<double> host((size_t)b->nrep * nv);
    BHIP(hipMemcpyAsync(host.data(), out, host.size() * sizeof(double), hipMemcpyDeviceToHost, st));
    BHIP(hipStreamSynchronize(st));
    for (int r = 0; r < b->nrep; ++r)
        for (int a = 0; a < b->q; ++a) {
            if (mode_sum) mode_sum[r * b->q + a] = host[(size_t)r * nv + a];
            if (mode_sumsq) mode_sumsq[r * b->q + a] = host[(size_t)r * nv + b->q + a];
        }
    if (nsamples) *nsamples = b->nsamples;
    for (double v : host)
        if (!std::isfinite(v)) return bfail(FLB_ERR_NONFINITE, "statistics are not finite");
    return FLB_OK;
}

flb_status flb_batch_reset_stats(flb_batch* b, void* stream) {
    if (!b) return bfail(FLB_ERR_INVALID_ARG, "batch is NULL");
    // the per-tile table is clear between calls; the accumulators follow it
    BHIP(launch_fill_zero(batch_acc(b), (size_t)b->nrep * 2 * b->q * sizeof(double),
                          (hipStream_t)stream));
    b->nsamples = 0;
    return FLB_OK;
}

flb_status flb_batch_state(const flb_batch* b, void** cur, void** other, uint64_t* step) {
    if (!b) return bfail(FLB_ERR_INVALID_ARG, "batch is NULL");
    if (cur) *cur = b->cur();
    if (other) *other = b->other();
    if (step) *step = b->step;
    return FLB_OK;
}

flb_status flb_batch_graph_capture(flb_batch* b, int64_t nsteps, int32_t stats_stride,
                                   void* stream) {
    if (!b) return bfail(FLB_ERR_INVALID_ARG, "batch is NULL");
    if (nsteps <= 0 || nsteps % 2 != 0 || stats_stride < 0)
        return bfail(FLB_ERR_INVALID_ARG, "graph step count must be positive and even");
    hipStream_t st = (hipStream_t)stream;
    if (!st) return bfail(FLB_ERR_INVALID_ARG, "graph capture needs a non-null stream");
    release_batch_graphs(b);
    // one recording for each buffer the state can be in (see flb_graph_capture)
    const bool cur_a = b->cur_a;
    int64_t ns = 0;
    flb_status r = FLB_OK;
    for (int k = 0; k < 2 && r == FLB_OK; ++k) {
        b->cur_a = k == 1;
        hipError_t e = hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess) {
            r = bfail(FLB_ERR_HIP, "begin capture: %s", hipGetErrorString(e));
            break;
        }
        r = batch_run(b, nsteps, stats_stride, true, st, &ns);
        hipGraph_t g = nullptr;
        e = hipStreamEndCapture(st, &g);
        if (r == FLB_OK && e != hipSuccess)
            r = bfail(FLB_ERR_HIP, "capture: %s", hipGetErrorString(e));
        if (r != FLB_OK) {
            if (g) (void)hipGraphDestroy(g);
            break;
        }
        b->graph[k] = g;
        e = hipGraphInstantiate(&b->gexec[k], g, nullptr, nullptr, 0);
        if (e != hipSuccess) r = bfail(FLB_ERR_HIP, "graph instantiate: %s", hipGetErrorString(e));
    }
    b->cur_a = cur_a;   // nothing ran
    if (r != FLB_OK) {
        release_batch_graphs(b);
        return r;
    }
    b->graph_steps = nsteps;
    b->graph_samples = ns;
    return FLB_OK;
}

flb_status flb_batch_graph_launch(flb_batch* b, void* stream) {
    if (!b) return bfail(FLB_ERR_INVALID_ARG, "batch is NULL");
    hipGraphExec_t ex = b->gexec[b->cur_a ? 1 : 0];
    if (!ex) return bfail(FLB_ERR_STATE, "no graph captured");
    BHIP(hipGraphLaunch(ex, (hipStream_t)stream));
    b->step += (uint64_t)b->graph_steps;
    b->nsamples += b->graph_samples;
    return FLB_OK;
}

flb_status flb_batch_autotune(flb_batch* b, int32_t repeats, int32_t* best, double* best_ms,
                              void* stream) {
    if (!b) return bfail(FLB_ERR_INVALID_ARG, "batch is NULL");
    if (repeats < 1) repeats = 1;
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t e0, e1;
    BHIP(hipEventCreate(&e0));
    BHIP(hipEventCreate(&e1));
    float bt[2] = {0.f, 0.f};
    // statistics trials only add to the per-tile table, cleared below; the
    // accumulators are not touched
    for (int mode = 0; mode < 2; ++mode) {
        double* part = mode ? b->stats : nullptr;
        const BatchGroup all = batch_all(b);
        BHIP(batch_one(b, 0, all, b->cur(), b->other(), nullptr, b->step, part, st));
        BHIP(hipEventRecord(e0, st));
        for (int r = 0; r < repeats; ++r)
            BHIP(batch_one(b, 0, all, b->cur(), b->other(), nullptr, b->step, part, st));
        BHIP(hipEventRecord(e1, st));
        BHIP(hipEventSynchronize(e1));
        BHIP(hipEventElapsedTime(&bt[mode], e0, e1));
        bt[mode] /= repeats;
    }
    // in-place pairs group by group, with statistics: the trials run in place
    // on a copy of the state in the other buffer (the next ordinary step
    // overwrites it), so the state is untouched
    if (b->nrep > 0) {
        BHIP(hipMemcpyAsync(b->other(), b->cur(), b->L.elems * b->rb, hipMemcpyDeviceToDevice,
                            st));
        uint64_t best_bytes = 0;
        float best_pair = bt[1];
        for (uint64_t mib : {64ull, 128ull, 160ull, 192ull, 224ull, 256ull, 320ull}) {
            const std::vector<BatchGroup> groups = batch_groups(b, mib << 20);
            BHIP(hipEventRecord(e0, st));
            for (const BatchGroup& G : groups)
                for (int j = 0; j < 2 * repeats; ++j)
                    BHIP(batch_one(b, 1 + (j & 1), G, b->other(), b->other(), nullptr, b->step + j,
                                   b->stats, st));
            BHIP(hipEventRecord(e1, st));
            BHIP(hipEventSynchronize(e1));
            float ms = 0.f;
            BHIP(hipEventElapsedTime(&ms, e0, e1));
            ms /= 2 * repeats;
            if (ms < best_pair) {
                best_pair = ms;
                best_bytes = mib << 20;
            }
        }
        b->pair_bytes = best_bytes;
        // the statistics trials added to the per-tile slots, which are clear
        // between calls: clear them again
        BHIP(launch_fill_zero(b->stats, (size_t)b->ntiles * 2 * b->q * sizeof(double), st));
        BHIP(hipStreamSynchronize(st));
        b->groups = best_bytes ? batch_groups(b, best_bytes) : std::vector<BatchGroup>();
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    for (int m = 0; m < 2; ++m) {
        if (best) best[m] = 0;   // one grid: a block per tile
        if (best_ms) best_ms[m] = bt[m];
    }
    return FLB_OK;
}

flb_status flb_batch_set_pairs(flb_batch* b, uint64_t pair_bytes) {
    if (!b) return bfail(FLB_ERR_INVALID_ARG, "batch is NULL");
    b->pair_bytes = pair_bytes;
    b->groups = pair_bytes ? batch_groups(b, pair_bytes) : std::vector<BatchGroup>();
    return FLB_OK;
}
flb_status flb_batch_pairs(const flb_batch* b, uint64_t* pair_bytes, int32_t* ngroups) {
    if (!b) return bfail(FLB_ERR_INVALID_ARG, "batch is NULL");
    if (pair_bytes) *pair_bytes = b->pair_bytes;
    if (ngroups) *ngroups = (int32_t)b->groups.size();
    return FLB_OK;
}
flb_status flb_batch_destroy(flb_batch* b) {
    if (!b) return FLB_OK;
    release_batch_graphs(b);
    delete b;
    return FLB_OK;
}

}  // extern "C"
