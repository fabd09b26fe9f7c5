// Several D2Q9 steps in one launch, for lattices that leave the chip idle.
//
// On a small lattice (128^2: 256 wavefronts) a step is a chain of latencies:
// launch, loads of populations that other XCDs wrote, a few hundred dependent
// operations, stores; 4.5 us at 128^2 with the vector units busy a fifth of
// that.  Here a block owns a tile of TX x TY sites and takes it through T
// steps: step s is computed on the tile plus a halo of H (T - 1 - s) sites, H
// the reach of one step (1 for the ideal gas; 3 with the force: a pull, the
// density, the chemical potential), and its populations stay in LDS for step
// s + 1.  Only step 0 reads global memory and only step T - 1 writes it, so T
// steps pay for one launch and one round trip.  The halo sites are computed by
// several blocks, from the same values with the same operations and noise
// counters, so the result has the bits of T ordinary steps.  The noise of all
// T steps is drawn while step 0's loads are in flight.
//
// It pays while the chip has lanes to spare (multi_steps); a large lattice
// is bound by issue or memory, where the halo is pure cost.
#pragma once
#include <hip/hip_runtime.h>

#include "device.h"
#include "internal.h"

namespace flb {

namespace {

// What a launch writes besides the last state: per step, its statistics
// (mask bit s: step s is sampled), the state it ends in (out[s], the last one
// always set) and the density it starts from (rho[s]); null: not wanted.
template <typename Real>
struct MultiOut {
    Real* out[MULTI_MAX];
    Real* rho[MULTI_MAX];
    uint32_t mask;
};

template <bool FORCE, int T, int TX, int TY>
struct MultiTile {
    static constexpr int H = FORCE ? 3 : 1;
    static constexpr int w(int s) { return TX + 2 * H * (T - 1 - s); }
    static constexpr int h(int s) { return TY + 2 * H * (T - 1 - s); }
    static constexpr int NT = (w(0) * h(0) + 63) / 64 * 64;
    // populations of the even and of the odd steps but the last
    static constexpr int NS0 = T > 1 ? 9 * w(0) * h(0) : 1;
    static constexpr int NS1 = T > 2 ? 9 * w(1) * h(1) : 1;
};

// Step S of the launch on its region of w x h sites; thread l has the site
// (l % w, l / w) if l < w h.
template <typename Real, bool FORCE, bool STATS, int T, int TX, int TY, int S>
struct MultiStep {
    using L = Lattice<0>;
    using MT = MultiTile<FORCE, T, TX, TY>;
    using M = Moments<0, Real>;
    static constexpr int W = MT::w(S), HH = MT::h(S), N = W * HH, Q = L::Q, NT = MT::NT;
    static constexpr int B = MT::H * (T - 1 - S);   // halo around the tile
    using FT = ForceTile<0, Real, W, HH, 1>;

    // the tile's site of this thread's place, wrapped into the box
    static __device__ __forceinline__ bool place(const Geom& g, int x0, int y0, int& lx, int& ly,
                                                 int& x, int& y) {
        const int l = (int)threadIdx.x;
        ly = l / W;
        lx = l - ly * W;
        x = wrap_any(x0 - B + lx, g.nx);
        y = wrap_any(y0 - B + ly, g.ny);
        return l < N;
    }
    static __device__ __forceinline__ void draw(const Geom& g, int x0, int y0, uint32_t step,
                                                const CollideParams<Real>& P, const double2* tab,
                                                Real (&zn)[2 * L::NPAIR]) {
        int lx, ly, x, y;
        if (!place(g, x0, y0, lx, ly, x, y) || !P.noise_on) return;
        site_normals<L::NPAIR, Real>(site_index<0>(x, y, 0, g), step + S, 0u, P.replica, P.key0,
                                     P.key1, zn, tab);
    }
    // f: the site's streamed populations; src (S > 0): the LDS populations of
    // step S - 1, whose region is H sites wider; dst: this step's (S < T - 1)
    static __device__ __forceinline__ void run(const Geom& g, int x0, int y0,
                                               const CollideParams<Real>& P,
                                               const ForceParams<Real>& fp, const Real* src,
                                               Real* dst, Real* rs, Real* ms, Real (&f)[Q],
                                               const Real* zn, const MultiOut<Real>& o, double* v) {
        constexpr int PW = W + 2 * MT::H, PN = PW * (HH + 2 * MT::H);
        int lx, ly, x, y;
        const bool in = place(g, x0, y0, lx, ly, x, y);
        auto pulled = [&](int px, int py, Real (&h)[Q]) {   // at place (px, py) of src's region
#pragma unroll
            for (int i = 0; i < Q; ++i) h[i] = src[i * PN + (py - L::cy[i]) * PW + px - L::cx[i]];
        };
        if constexpr (S > 0) {
            if (in) pulled(lx + MT::H, ly + MT::H, f);
            if constexpr (FORCE) {
                for (int l = threadIdx.x; l < FT::NR; l += NT) {
                    const int ry = l / FT::RX, rx = l - ry * FT::RX;
                    Real h[Q], acc = Real(0);
                    pulled(rx + MT::H - 2, ry + MT::H - 2, h);
#pragma unroll
                    for (int i = 0; i < Q; ++i) acc += h[i];
                    rs[l] = acc;
                }
                __syncthreads();
            }
        }
        Real F[2] = {Real(0), Real(0)};
        if constexpr (FORCE) {
            FT::mu_from_rho(fp, rs, ms, NT);   // ends with a barrier
            if (in) FT::force(rs, ms, fp, P.rho0, lx, ly, 0, F);
        }
        if (!in) return;
        const bool own = lx >= B && lx < B + TX && ly >= B && ly < B + TY && x0 - B + lx < g.nx &&
                         y0 - B + ly < g.ny;
        const uint32_t site = site_index<0>(x, y, 0, g);
        if (own && o.rho[S]) {
            Real acc = Real(0);
#pragma unroll
            for (int i = 0; i < Q; ++i) acc += f[i];
            o.rho[S][site] = acc;
        }
        Real m[Q];
        M::forward(f, m);
        if constexpr (STATS) {
            if (own && ((o.mask >> S) & 1u)) {
#pragma unroll
                for (int a = 0; a < Q; ++a) {
                    v[a] += m[a];
                    v[Q + a] += (double)m[a] * (double)m[a];
                }
            }
        }
        collide_moments<0, Real, FORCE>(m, F, zn, P);
        M::inverse(m, f);
        if constexpr (S + 1 < T) {
#pragma unroll
            for (int i = 0; i < Q; ++i) dst[i * N + (int)threadIdx.x] = f[i];
        }
        if (own && o.out[S]) {
#pragma unroll
            for (int i = 0; i < Q; ++i) plane_st(o.out[S] + (size_t)i * g.V, site, f[i]);
        }
    }
};

template <typename Real, bool FORCE, bool STATS, int T, int TX, int TY>
__global__ __launch_bounds__((MultiTile<FORCE, T, TX, TY>::NT)) void k_multi(
    const Real* __restrict__ fin, Geom g, CollideParams<Real> P, ForceParams<Real> fp, StepIndex st,
    double* __restrict__ partial, MultiOut<Real> o) {
    using L = Lattice<0>;
    using MT = MultiTile<FORCE, T, TX, TY>;
    using S0 = MultiStep<Real, FORCE, STATS, T, TX, TY, 0>;
    using FT = typename S0::FT;
    constexpr int Q = L::Q, NT = MT::NT, Z = 2 * L::NPAIR;
    __shared__ Real s0[MT::NS0];
    __shared__ Real s1[MT::NS1];
    __shared__ Real rs[FORCE ? FT::NR : 1];
    __shared__ Real ms[FORCE ? FT::NM : 1];
    __shared__ double lds_stats[STATS ? 4 * (NT / 64) * 2 * Q : 1];
    int x0, y0, z0;
    tile_origin<0, TX, TY, 1>(g, x0, y0, z0);

    // step 0's loads: the thread's site and, with the force, a site of the
    // two-wide ring around the region whose density is needed
    int lx, ly, x, y;
    const bool in = S0::place(g, x0, y0, lx, ly, x, y);
    constexpr int NRING = FORCE ? FT::NR - S0::N : 0;
    auto ring_at = [&](int r, int& rx, int& ry) {
        if (r < 4 * FT::RX) {
            const int k = r / FT::RX;   // rows 0, 1, RY - 2, RY - 1
            rx = r - k * FT::RX;
            ry = k < 2 ? k : FT::RY - 4 + k;
        } else {
            const int c = r - 4 * FT::RX, k = c / S0::HH;   // columns 0, 1, RX - 2, RX - 1
            rx = k < 2 ? k : FT::RX - 4 + k;
            ry = 2 + (c - k * S0::HH);
        }
    };
    static_assert(NRING <= NT, "a ring site per thread at most");
    Real f[Q], h[FORCE ? Q : 1];
    int rx = 0, ry = 0;
    if (in) pull<0, Real>(fin, x, y, 0, g, f);
    if constexpr (FORCE) {
        if ((int)threadIdx.x < NRING) {
            ring_at((int)threadIdx.x, rx, ry);
            pull<0, Real>(fin, wrap_any(x0 - S0::B + rx - 2, g.nx),
                          wrap_any(y0 - S0::B + ry - 2, g.ny), 0, g, h);
        }
    }
    const double2* tab = noise_table<Real, NT>();
    const uint32_t step = st.get();
    Real z[T][Z];
    S0::draw(g, x0, y0, step, P, tab, z[0]);
    if constexpr (T > 1) MultiStep<Real, FORCE, STATS, T, TX, TY, 1>::draw(g, x0, y0, step, P, tab, z[1]);
    if constexpr (T > 2) MultiStep<Real, FORCE, STATS, T, TX, TY, 2>::draw(g, x0, y0, step, P, tab, z[2]);
    if constexpr (T > 3) MultiStep<Real, FORCE, STATS, T, TX, TY, 3>::draw(g, x0, y0, step, P, tab, z[3]);
    if constexpr (FORCE) {
        if (in) {
            Real acc = Real(0);
#pragma unroll
            for (int i = 0; i < Q; ++i) acc += f[i];
            rs[(ly + 2) * FT::RX + lx + 2] = acc;
        }
        if ((int)threadIdx.x < NRING) {
            Real acc = Real(0);
#pragma unroll
            for (int i = 0; i < Q; ++i) acc += h[i];
            rs[ry * FT::RX + rx] = acc;
        }
        __syncthreads();
    }
    // Statistics: a thread adds its steps in FP64, as steps of a launch of their
    // own are (an FP32 sum over the steps dropped what is below 2^-24 of it), with
    // one reduction for all of them: 200 x 200 FP32, ideal gas, 2.36 -> 2.44 us a
    // step, Landau 3.97 -> 4.05 (one step per launch 3.9 and 5.4); the rows of
    // every step reduced to FP64 by themselves took 2.54 and 4.06.
    double v[STATS ? 2 * Q : 1];
#pragma unroll
    for (int k = 0; k < (STATS ? 2 * Q : 1); ++k) v[k] = 0.0;
    // between two steps a barrier: the populations just written are read, and
    // the density and chemical potential just read are overwritten
    S0::run(g, x0, y0, P, fp, nullptr, s0, rs, ms, f, z[0], o, v);
    if constexpr (T > 1) {
        __syncthreads();
        MultiStep<Real, FORCE, STATS, T, TX, TY, 1>::run(g, x0, y0, P, fp, s0, s1, rs, ms, f, z[1], o, v);
    }
    if constexpr (T > 2) {
        __syncthreads();
        MultiStep<Real, FORCE, STATS, T, TX, TY, 2>::run(g, x0, y0, P, fp, s1, s0, rs, ms, f, z[2], o, v);
    }
    if constexpr (T > 3) {
        __syncthreads();
        MultiStep<Real, FORCE, STATS, T, TX, TY, 3>::run(g, x0, y0, P, fp, s0, s1, rs, ms, f, z[3], o, v);
    }
    if constexpr (STATS) {
        const uint32_t b = xcd_remap(blockIdx.x, g.nblocks);
        block_accumulate<2 * Q, NT>(v, partial + (size_t)b * 2 * Q, lds_stats);
    }
}

}  // namespace
}  // namespace flb
